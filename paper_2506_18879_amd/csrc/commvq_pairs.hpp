// Paired-code keys (App. A.1), the paper's own key format: table re-layout and score kernel (included by commvq.hip).
#pragma once

namespace {

// Per token and KV head R residual levels, each a pair (a, b) of 6-bit
// indices into ONE table of N_c' = 64 centres per level; level r contributes C[r][a] + i C[r][b]
// (Eq. def_center: per 2-D sub-space (x_a - y_b, y_a + x_b)), i.e. index form with 2R tied codebooks.
constexpr int kPairK = 64;       // centres per level
constexpr int kPairPlanes = 4;   // 8-element planes per LDS slice (4 slices cover the 16 planes of d = 128)
constexpr int kPairSet = kPairK * 256;    // bytes of a set of four levels: 64 rows x 16 pieces

// Tied table [Hkv][R][64][d] bf16 -> LDS images for k_score_pair:
//   packed[g][slice][set][c][4 plane + k] 16-byte pieces = elements 8 (4 slice + plane) .. +7 of centre c of
//   level 4 set + k (zeros for levels >= R).  One thread per piece of the output.
__global__ __launch_bounds__(256) void k_prep_pairs(const uint4 *__restrict__ table, uint4 *__restrict__ packed, int Hkv,
                                                    int R, int sets)
{
    const size_t n = (size_t)Hkv * 4 * sets * kPairK * 16;
    const size_t t = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= n) return;
    const int col = (int)(t & 15);
    const int c = (int)((t >> 4) % kPairK);
    size_t rest = (t >> 4) / kPairK;
    const int set = (int)(rest % sets);
    rest /= sets;
    const int slice = (int)(rest % 4), g = (int)(rest / 4);
    const int r = 4 * set + (col & 3);
    uint4 v = make_uint4(0, 0, 0, 0);
    if (r < R) v = table[(((size_t)g * R + r) * kPairK + c) * 16 + 4 * slice + (col >> 2)];
    packed[t] = v;
}

// Score kernel for paired-code keys: k_score_stream (which see for tokens, segments, the contraction and the write-out) with another gather.  Differences:
//   * A slice = 4 planes of 8 elements of every centre of every level, SETS sets of four levels: a set is 64 rows (centre
//     index) of 16 bank columns, 4 of them per plane.  A plane takes the place of a slice there: four rounds per slice.
//   * Lanes n with the same n / 4 = j work on plane i ^ j in round i.  The four lanes of a token are (a | b) x half: in step (s, st)
//     lane (n, g) gathers, for its tokens of both sets of 16, the centre that the a (g even) or b index selects in level
//     4 s + (n + 2 (g >> 1) + st) mod 4.  The 16 lanes that a 16-byte read checks against each other
//     are four such quads with four different j (0..3, 12..15, 20..23, 24..27 of every 32 lanes, and the other 16): four planes
//     x four levels, 16 bank columns whatever the indices.
//   * The selection operand adds a pieces as they are and b pieces as i C[b] = (-y, x): element e ^ 1, negated for x.
//   * The 12-bit pairs are taken apart here, once per tile: lane (n, g) reads the record of its token of set g >> 1 and makes
//     index bytes of one type of all levels, the two halves of the wavefront exchange them, and a byte permute per pair of
//     sets leaves the bytes of the lane's own steps, which stay in registers.
//     (Buffer loads check each dword against the end of the stream by itself.)
//   * Phase factors and queries of a slice (four times those of one plane) come through registers, requested in the last
//     round of the slice before.
// What bounds it: SIMD issue and LDS as there, 6 (12) sparse matrix instructions, 12 (24) byte permutes, 5 products and a rotation of 8
// per 32 tokens and plane for R = 11 (21) and 4 heads (with the exchange of rows instead of logits in halves: paper's 1-bit setting at 128K
// 112.4 us a call, 107.7 so).  Whole calls with binary values, before (index bytes unpacked
// by a kernel of their own, 17 us at 128K, and read again for every slice; columns for 16 or 32 levels; totals over lanes; tiles
// of one sequence, never cut along the planes) and now, R = 11 | 21: 2000 tokens 58.3 -> 39.7 | 78.5 -> 42.6 us, 12000 59.6 ->
// 48.2 | 81.1 -> 56.3, 40000 84.1 -> 74.4 | 125.8 -> 89.2, 128K 146.8 -> 117.3 | 250 -> 197, 8 x 1100..2200 63.1 -> 55.9 | 84.3 -> 62.2.
// With two groups of heads the most passes do not fit the registers: <3, 2, 8> spills 22 of them, <6, 2, 6> 38.
template <int SETS, int FORM, int NP>
__global__ __launch_bounds__(kSliceThreads) void k_score_pair(
    const void *__restrict__ q, const uint8_t *__restrict__ pairs, const uint4 *__restrict__ packed,
    const int32_t *__restrict__ cu, const int32_t *__restrict__ q_pos, const float2 *__restrict__ tbl_hi,
    const float2 *__restrict__ tbl_lo, float *__restrict__ scores, float2 *__restrict__ sstat, const StreamDims a, const int R, const int PB)
{
    constexpr int S = kPairSlices, PL = kPairPlanes;
    constexpr int NST = 2 * SETS;                             // gather steps (sparse matrix instructions) per pass
    constexpr bool TWO = SETS == 3;                           // slices in two LDS buffers in turn, else in one
    constexpr int NGRP = FORM == 2 ? 2 : 1;                   // (FORM as for k_score_stream)
    const int G = NGRP == 2 ? 8 : a.G;                        // query heads of the KV head; NGRP groups of 4, padded with zero queries
    constexpr int NBUF = 2;                                   // gather steps whose LDS reads are in flight
    constexpr bool HALF = FORM == 1;
    constexpr int CC = SETS == 3 ? 3 : SETS;                  // dwords of a lane's index bytes per pass
    constexpr int RAW = SETS == 3 ? 5 : SETS == 4 ? 7 : 8;    // dwords that hold a record at any byte offset
    // LDS: slice buffers at 0 (and 64 KiB), [8 parts][64 positions] fine factors, queries, coarse factors [pass][9 rows][8 parts, padded
    // to 12: the four rows of a quad are then 4 entries apart mod 16, its part another mod 4], and what the write-out needs
    constexpr int HROW = 12, ELO_AT = SETS == 6 ? 98304 : SETS == 4 ? 65536 : 49152, Q_AT = ELO_AT + 8192, EHI_AT = SETS == 3 ? 114688 : Q_AT + 8192;
    constexpr int SEG_AT = EHI_AT + kStreamPasses * kHiRows * HROW * 16, DIST_AT = SEG_AT + kStreamPasses * 16, WST_AT = DIST_AT + kStreamPasses * 4;
    static_assert(WST_AT + kStreamPasses * 2 * 8 * 8 <= kPairLds && 4 * NP * 8 * 68 * 4 <= SEG_AT, "LDS layout");
    extern __shared__ __attribute__((aligned(16))) uint4 tab[];

    int id = blockIdx.x;
    const int g = id % a.Hkv;                                 // (head = index mod Hkv: with 8 KV heads an XCD serves one head)
    id /= a.Hkv;
    const int tile = id % a.tiles;
    const int eg = id / a.tiles;                              // which group of rounds (a slice's planes, each in another lane, or all of it)
    const int r_begin = eg * (S * PL / a.groups), r_end = r_begin + S * PL / a.groups, s_begin = r_begin / PL, s_end = (r_end + PL - 1) / PL;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    const char *src = reinterpret_cast<const char *>(packed) + (size_t)g * S * SETS * kPairSet;
    auto send_set = [&](int sl, int set) {
        const char *p = src + ((size_t)sl * SETS + set) * kPairSet;
        lds_dma16(p, (unsigned)(wave * 64 + fresh_lane()) * 16u, (unsigned)((TWO ? (sl & 1) * 65536 : 0) + set * kPairSet + wave * 1024));
    };
#pragma unroll
    for (int k = 0; k < SETS; ++k) send_set(s_begin, k);

    // This workgroup's segments: pass p works on tokens pt0[p] .. + 511 of sequence pb[p].  Every wavefront finds them by
    // itself, 64 sequences at a time (prefix sums of the sequences' segment counts).
    int pb[NP], pt0[NP], pL[NP], pcu[NP];
    int qd[NP];                                               // distance of the segment's first token to its query
    int np = 0;                                               // passes that exist
#pragma unroll
    for (int p = 0; p < NP; ++p) { pb[p] = 0; pt0[p] = 0; pL[p] = 0; pcu[p] = 0; qd[p] = 0; }
    const int first = tile * NP;
    if (a.batch == 1) {
        const int c0 = cu[0], L = cu[1] - c0, qp = q_pos[0];
#pragma unroll
        for (int p = 0; p < NP; ++p) { pt0[p] = (first + p) * kPassTokens; pL[p] = L; pcu[p] = c0; qd[p] = qp - pt0[p]; }
        np = min(NP, (L + kPassTokens - 1) / kPassTokens - first);
    } else {
        int before = 0;                                       // segments of the sequences before this round of 64
        for (int c = 0; c < a.batch; c += 64) {
            const int bb = c + lane;
            const int c0 = bb < a.batch ? cu[bb] : 0, Lb = bb < a.batch ? cu[bb + 1] - c0 : 0, qp = bb < a.batch ? q_pos[bb] : 0;
            const int nb = (Lb + kPassTokens - 1) / kPassTokens;
            int incl = nb;
#pragma unroll
            for (int d = 1; d < 64; d *= 2) {
                const int t = __shfl_up(incl, d);
                if (lane >= d) incl += t;
            }
            const int start = before + incl - nb;
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const int s = first + p;
                const unsigned long long hit = __ballot(s >= start && s < start + nb);
                if (hit) {
                    const int l = __builtin_ctzll(hit);
                    pb[p] = c + l;
                    pt0[p] = (s - __builtin_amdgcn_readlane(start, l)) * kPassTokens;
                    pL[p] = __builtin_amdgcn_readlane(Lb, l);
                    pcu[p] = __builtin_amdgcn_readlane(c0, l);
                    qd[p] = __builtin_amdgcn_readlane(qp, l) - pt0[p];
                    np = p + 1;
                }
            }
            before += __builtin_amdgcn_readlane(incl, 63);
            if (before >= first + NP) break;
        }
    }
    if (np <= 0) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // the sets sent for above have landed
        return;
    }
    unsigned chg = 1u;                                        // bit p: pass p is of another sequence than pass p - 1
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        if (p > 0 && p < np && pb[p] != pb[p - 1]) chg |= 1u << p;
    }

    const int n = lane & 15, gk = lane >> 4;
    const int par = gk & 1, hi = gk >> 1;                     // par: half of the 8 elements; hi: set of 16 tokens
    const int f = 4 * wave + (n >> 2);                        // fine position

    // The records: lane (n, gk) reads that of its token of set hi and takes the indices of type par (0: a, 1: b) out of it.  (The
    // descriptor begins at the aligned dword below the stream and ends with the dword that holds its last byte: tokens past the end
    // read zeros, index 0 of every level.)
    unsigned ccall[NP][CC];
    {
        unsigned raw[NP][RAW], sh[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const uintptr_t first = reinterpret_cast<uintptr_t>(pairs) + ((size_t)pcu[p] * a.Hkv + (size_t)g * pL[p]) * PB;
            const unsigned skew = (unsigned)(first & 3u);
            const __amdgpu_buffer_rsrc_t rs = make_rsrc(reinterpret_cast<const void *>(first - skew), p < np ? (skew + (unsigned)pL[p] * (unsigned)PB + 3u) & ~3u : 0u);
            const unsigned at = skew + (unsigned)(pt0[p] + f + kLo * ((n & 3) + 4 * hi)) * (unsigned)PB;
            sh[p] = (at & 3u) * 8u + 6u * par;
            const uint4_t c = __builtin_amdgcn_raw_buffer_load_b128(rs, at & ~3u, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) raw[p][i] = c[i];
            if constexpr (RAW == 5) {
                raw[p][4] = __builtin_amdgcn_raw_buffer_load_b32(rs, (at & ~3u) + 16u, 0, 0);
            } else {
                const uint4_t d = __builtin_amdgcn_raw_buffer_load_b128(rs, (at & ~3u) + 16u, 0, 0);
#pragma unroll
                for (int i = 4; i < RAW; ++i) raw[p][i] = d[i - 4];
            }
        }
        const unsigned b0 = (unsigned)(n + 2 * hi) & 3u, b1 = (unsigned)(n + 2 * hi + 1) & 3u;
        const unsigned own = b0 | b1 << 8 | (4u + b0) << 16 | (4u + b1) << 24;  // bytes of the lane's steps of two sets
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            unsigned win[RAW + 2];                            // the record from the first index of the lane's type on
#pragma unroll
            for (int i = 0; i < RAW; ++i) win[i] = __builtin_amdgcn_alignbit(i + 1 < RAW ? raw[p][i + 1] : 0u, raw[p][i], sh[p]);
            win[RAW] = win[RAW + 1] = 0u;
            unsigned d[2][SETS];                              // both sets' tokens: a dword of four levels
#pragma unroll
            for (int s = 0; s < SETS; ++s) {
                const int dw = 48 * s >> 5;
                const unsigned lo = s & 1 ? __builtin_amdgcn_alignbit(win[dw + 1], win[dw], 16) : win[dw];
                const unsigned up = s & 1 ? __builtin_amdgcn_alignbit(win[dw + 2], win[dw + 1], 16) : win[dw + 1];
                unsigned w = (lo & 63u) | (lo >> 4 & 0x3f00u) | (lo >> 8 & 0x3f0000u) | (up << 20 & 0x3f000000u);
                if (4 * s + 4 > R) w &= 4 * s >= R ? 0u : 0xffffffffu >> (8 * (4 * s + 4 - R));
                auto r = __builtin_amdgcn_permlane32_swap(w, w, false, false);  // lower half of the wavefront: set 0, upper half: set 1
                d[0][s] = r[0];
                d[1][s] = r[1];
            }
            if constexpr (SETS == 3) {
                ccall[p][0] = __builtin_amdgcn_perm(d[0][1], d[0][0], own);
                ccall[p][1] = __builtin_amdgcn_perm(d[1][1], d[1][0], own);
                ccall[p][2] = __builtin_amdgcn_perm(d[1][2], d[0][2], own);
            } else {
#pragma unroll
                for (int v = 0; v < 2; ++v)
#pragma unroll
                    for (int k = 0; k < SETS / 2; ++k) ccall[p][v * (SETS / 2) + k] = __builtin_amdgcn_perm(d[v][2 * k + 1], d[v][2 * k], own);
            }
        }
    }

    // the segments, for phase factors, queries and the write-out
    int4 *segs_w = reinterpret_cast<int4 *>(reinterpret_cast<char *>(tab) + SEG_AT);
    int *dist_w = reinterpret_cast<int *>(reinterpret_cast<char *>(tab) + DIST_AT);
    if (wave == 0 && lane < NP) {
        int4 s = make_int4(0, 0, 0, 0);
        int D = 0;
#pragma unroll
        for (int p = 0; p < NP; ++p)
            if (lane == p) { s = make_int4(pb[p], pt0[p], pL[p], pcu[p]); D = qd[p]; }
        segs_w[lane] = s;
        dist_w[lane] = D;
    }
    __syncthreads();

    // What a slice needs besides the table, two pieces of 16 bytes per thread: fine factors [8 parts][64], coarse ones
    // [pass][9 rows][8 parts], queries [pass][head][32 elements].
    const int per = a.q_bf16 ? 4 : 8;
    uint4_t aux[2];
    auto aux_load = [&](int sl) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int x = k * kSliceThreads + wave * 64 + fresh_lane(), y = x - 8 * kLo, z = y - NP * kHiRows * 8;
            const char *p = nullptr;
            bool flip = false;
            if (y < 0) {
                p = reinterpret_cast<const char *>(tbl_lo + (size_t)(x % kLo) * kJ + 16 * sl + 2 * (x / kLo));
            } else if (z < 0) {
                const int row = y >> 3, pass = row / kHiRows;
                const int H = ((dist_w[pass] + 1) >> kLoBits) - 8 + row % kHiRows;  // rows 0..8: what distances D - 511 .. D can reach
                flip = H < 0;                                 // the conjugate of the row of |H|
                p = reinterpret_cast<const char *>(tbl_hi + (size_t)min(flip ? -H : H, a.n_hi - 1) * kJ + 16 * sl + 2 * (y & 7));
            } else if (z < NP * G * per) {
                const int pass = z / (G * per), h = z / per % G;
                p = static_cast<const char *>(q) + (((size_t)segs_w[pass].x * a.Hq + (size_t)g * G + h) * kD + 32 * sl) * (a.q_bf16 ? 2 : 4) + z % per * 16;
            }
            uint4_t v = {0u, 0u, 0u, 0u};
            if (p) {
                typedef unsigned u4u __attribute__((ext_vector_type(4), aligned(2)));  // (queries may have any alignment that their elements have)
                const u4u w = *reinterpret_cast<const u4u *>(p);
                v = uint4_t{w[0], w[1], w[2], w[3]};
            }
            if (flip) { v[1] ^= 0x80000000u; v[3] ^= 0x80000000u; }
            aux[k] = v;
        }
    };
    auto aux_store = [&]() {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int x = k * kSliceThreads + wave * 64 + fresh_lane(), y = x - 8 * kLo, z = y - NP * kHiRows * 8;
            char *dst = reinterpret_cast<char *>(tab) + (y < 0 ? ELO_AT + x * 16 : z < 0 ? EHI_AT + ((y >> 3) * HROW + (y & 7)) * 16 : Q_AT + z * 16);
            if (z < NP * G * per) *reinterpret_cast<uint4_t *>(dst) = aux[k];
        }
    };
    aux_load(s_begin);

    // Selection operand of v_smfmac_f32_16x16x64_bf16 (layout: see k_score_stream).  First-operand lane (row i, block q) covers
    // the pieces of second-operand lanes 2 (q & 1) (type a: groups of four 0 and 1) and 2 (q & 1) + 1 (type b: groups 2 and 3), the
    // first piece for q < 2, the second for q >= 2; rows 0..7 add set 0's first pieces, rows 8..15 set 1's second ones.
    uint4_t sel = {0u, 0u, 0u, 0u};
    unsigned sidx = 0x44444444u;  // default positions (0, 1) of every stored pair
    {
        const int e = n & 7;
        if ((n < 8) == (gk < 2)) {
            const int t = e >> 2, pa = e & 3, pb2 = (e ^ 1) & 3;
            sel[t] = 0x00003f80u;                             // + element e of a
            sel[2 + t] = e & 1 ? 0x00003f80u : 0x0000bf80u;   // +- element e ^ 1 of b
            const unsigned ia = (unsigned)pa | (pa == 0 ? 4u : 0u), ib = (unsigned)pb2 | (pb2 == 0 ? 4u : 0u);
            sidx = (sidx & ~(0xfu << (4 * t)) & ~(0xfu << (4 * (2 + t)))) | ia << (4 * t) | ib << (4 * (2 + t));
            sidx = (sidx & 0xffffu) | sidx << 16;
        }
    }
    const bf16x8_t selv = __builtin_bit_cast(bf16x8_t, sel);

    constexpr int NPAIR = (NP + 1) / 2;
    // HALF: 4 heads of the lane's token of pass p, from the lane's half of the elements; else 4 heads of its token of pass 2 k + par
    constexpr int NV = HALF ? NP : NPAIR;
    floatx4_t sc[NV][NGRP];
#pragma unroll
    for (int k = 0; k < NV; ++k)
#pragma unroll
        for (int x = 0; x < NGRP; ++x) sc[k][x] = floatx4_t{0.f, 0.f, 0.f, 0.f};

    float zero = 0.f;
    asm volatile("" : "+v"(zero));
    uint4_t v[NBUF][2];
    float qrow[NGRP][HALF ? 4 : 8];                                      // q' of the plane: head 4 x + n % 4, the 8 elements
    unsigned ehi_at = 0u;                                     // LDS address of the lane's coarse factor in pass 0's rows
    // the lane's row among the coarse factors of a pass whose first token is D away from its query, and its part in round 0
    auto hi_row = [&](int D, int i) {
        const int ln = fresh_lane(), j = ln >> 2 & 3;
        const int row = ((D - 4 * wave - j) >> kLoBits) - ((D + 1) >> kLoBits) + 8 - (ln & 3) - 4 * (ln >> 5);
        ehi_at = (unsigned)EHI_AT + (unsigned)(row * HROW + 2 * (i ^ j) + (ln >> 4 & 1)) * 16u;
    };
    for (int sl = s_begin; sl < s_end; ++sl) {
        const bool more = sl + 1 < s_end;
        // everyone is done with what is overwritten now: the phase factors and queries, and the table where there is one buffer
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        bare_barrier();
        if (!TWO && sl > s_begin) {
#pragma unroll
            for (int k = 0; k < SETS; ++k) send_set(sl, k);
        }
        aux_store();
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        bare_barrier();
        const unsigned slot_sel = (unsigned)(2 + (sl & 1)) << 16;
#pragma unroll 1
        for (int i = max(r_begin - PL * sl, 0); i < min(r_end - PL * sl, PL); ++i) {
        // an opaque copy per round: the gather addresses made from these must not be hoisted out (they would
        // take several registers per pass)
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int k = 0; k < CC; ++k) asm volatile("" : "+v"(ccall[p][k]));
        unsigned xreg[2];
        {
            const int ln = fresh_lane();
#pragma unroll
            for (int st = 0; st < 2; ++st) xreg[st] = (unsigned)(4 * (i ^ (ln >> 2 & 3)) + ((ln + 2 * (ln >> 5) + st) & 3)) * 16u | 1u << 24;
        }
        auto issue = [&](int p, int st) {
            const int set = st / 2;
#pragma unroll
            for (int ab = 0; ab < 2; ++ab) {
                const int word = SETS == 3 ? (set < 2 ? ab : 2) : ab * (SETS / 2) + set / 2, byte = (SETS == 3 && set == 2 ? ab : set & 1) * 2 + (st & 1);
                const unsigned psel = 0x0c000000u | (unsigned)(4 + byte) << 8 | (TWO ? slot_sel : (unsigned)(2 + set / 4) << 16);
                v[(p * NST + st) % NBUF][ab] = lds_read_b128(__builtin_amdgcn_perm(ccall[p][word], xreg[st & 1], psel) + (unsigned)(set % 4 * kPairSet));
            }
        };
        // q' = q conj(E_lo) for the pair of passes k (Re(conj(q) a E_hi E_lo) = Re(conj(q') a E_hi))
        // HALF: for pass k, the lane's 4 elements
        auto fold = [&](int k) __attribute__((always_inline)) {
            const int ln = fresh_lane(), odd = ln >> 4 & 1, j = ln >> 2 & 3, pl = i ^ j;
            if constexpr (HALF) {
                const unsigned lo = (unsigned)ELO_AT + (unsigned)((2 * pl + odd) * kLo + ((qd[k] - 4 * wave - j) & (kLo - 1))) * 16u;
                const uint4_t e = lds_read_b128(lo);
                const int h = ln & 3;
                const unsigned at = (unsigned)Q_AT + (unsigned)((k * G + h) * per + (a.q_bf16 ? pl : 2 * pl)) * 16u + odd * (a.q_bf16 ? 8u : 16u);
                float qv[4];
                if (a.q_bf16) {
                    const uint2_t w = *reinterpret_cast<lds_u2_ptr>(at);
#pragma unroll
                    for (int r = 0; r < 2; ++r) {
                        const unsigned u = w[r];
                        qv[2 * r] = bf16_lo(u);
                        qv[2 * r + 1] = bf16_hi(u);
                    }
                } else {
                    const uint4_t w = lds_read_b128(at);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const unsigned u = w[r];
                        qv[r] = __builtin_bit_cast(float, u);
                    }
                }
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const unsigned lxr = e[2 * u], lyr = e[2 * u + 1];
                    const float lx = __builtin_bit_cast(float, lxr), ly = __builtin_bit_cast(float, lyr);
                    const float qx = qv[2 * u], qy = qv[2 * u + 1];
                    qrow[0][2 * u] = h >= G ? 0.f : qx * lx + qy * ly;
                    qrow[0][2 * u + 1] = h >= G ? 0.f : qy * lx - qx * ly;
                }
                return;
            }
            const int d0 = qd[2 * k % NP], d1 = qd[2 * k + 1 < NP ? 2 * k + 1 : 2 * k % NP], D = odd ? d1 : d0;
            const unsigned lo = (unsigned)ELO_AT + (unsigned)(2 * pl * kLo + ((D - 4 * wave - j) & (kLo - 1))) * 16u;
            const uint4_t e0 = lds_read_b128(lo), e1 = lds_read_b128(lo + kLo * 16u);
#pragma unroll
            for (int x = 0; x < NGRP; ++x) {
                const int h = 4 * x + (ln & 3);
                const unsigned at = (unsigned)Q_AT + (unsigned)(((2 * k + odd) * G + h) * per + (a.q_bf16 ? pl : 2 * pl)) * 16u;
                float qv[8];
                if (a.q_bf16) {
                    const uint4_t w = lds_read_b128(at);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const unsigned u = w[r];
                        qv[2 * r] = bf16_lo(u);
                        qv[2 * r + 1] = bf16_hi(u);
                    }
                } else {
                    const uint4_t w0 = lds_read_b128(at), w1 = lds_read_b128(at + 16u);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const unsigned u0 = w0[r], u1 = w1[r];
                        qv[r] = __builtin_bit_cast(float, u0);
                        qv[4 + r] = __builtin_bit_cast(float, u1);
                    }
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const unsigned lxr = u < 2 ? e0[2 * u] : e1[2 * u - 4], lyr = u < 2 ? e0[2 * u + 1] : e1[2 * u - 3];
                    const float lx = __builtin_bit_cast(float, lxr), ly = __builtin_bit_cast(float, lyr);
                    const float qx = qv[2 * u], qy = qv[2 * u + 1];
                    qrow[x][2 * u] = NGRP == 1 && h >= G ? 0.f : qx * lx + qy * ly;
                    qrow[x][2 * u + 1] = NGRP == 1 && h >= G ? 0.f : qy * lx - qx * ly;
                }
            }
        };
        // the lane's sub-space u (of two), rotated by the coarse phase factor: A E_hi
        auto rotate = [&](int u, const floatx4_t &acc, const uint4_t &eh, float *val) {
            const unsigned hxr = eh[2 * u], hyr = eh[2 * u + 1];
            const float ex = __builtin_bit_cast(float, hxr), ey = __builtin_bit_cast(float, hyr);
            const float ax = acc[2 * u], ay = acc[2 * u + 1];
            val[2 * u] = ax * ex - ay * ey;
            val[2 * u + 1] = ax * ey + ay * ex;
        };
        // 2. and 3. for pass p, in NST parts that run between the steps of the next pass
        float val[4];
        auto finish_half = [&](auto pc, const floatx4_t &acc, const uint4_t &eh, int st) __attribute__((always_inline)) {
            constexpr int p = decltype(pc)::value;
            if (st == 0) {
                rotate(0, acc, eh, val);
                rotate(1, acc, eh, val);
            } else {
#pragma unroll
                for (int r = (st - 1) * 4 / (NST - 1); r < st * 4 / (NST - 1); ++r)
                    sc[HALF ? p : 0][0] = __builtin_amdgcn_mfma_f32_4x4x1f32(qrow[0][r], val[r], sc[HALF ? p : 0][0], 0, 0, 0);
            }
        };
        floatx4_t acc_e, acc_o;                               // gather sums of the pair's even and odd pass
        uint4_t eh_e, eh_o;                                   // their coarse phase factors
        float xy[8];                                          // even pass: rotated elements in 0..3; then the lane's 8 elements
        // 2. and 3. for a pair of passes, in NST parts that run between the steps of the next pass
        auto finish = [&](int k, int st) {
            if (st == 0) {
                float odd[4];
                rotate(0, acc_o, eh_o, odd);
                rotate(1, acc_o, eh_o, odd);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    auto s = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, xy[r]), __builtin_bit_cast(unsigned, odd[r]), false, false);
                    const unsigned s0 = s[0], s1 = s[1];
                    xy[r] = __builtin_bit_cast(float, s0);
                    xy[4 + r] = __builtin_bit_cast(float, s1);
                }
            } else {
#pragma unroll
                for (int r = (st - 1) * 8 / (NST - 1); r < st * 8 / (NST - 1); ++r)
#pragma unroll
                    for (int x = 0; x < NGRP; ++x) sc[k][x] = __builtin_amdgcn_mfma_f32_4x4x1f32(qrow[x][r], xy[r], sc[k][x], 0, 0, 0);
            }
        };
        // 1. the gather-sum of pass p on the matrix cores, with a part of other work after every step
        auto pass = [&](auto pc, floatx4_t &acc, uint4_t &eh, auto part) __attribute__((always_inline)) {
            constexpr int p = decltype(pc)::value;
            __builtin_amdgcn_sched_barrier(0);
            // (wavefronts that are behind go first; pass by pass towards the barrier, where a last one would be alone on its SIMD)
            __builtin_amdgcn_s_setprio(p < NP - 4 ? 3 : p < NP - 2 ? 2 : NP - 1 - p);
            if (p == 0 || __builtin_expect(chg >> p & 1u, 0)) hi_row(qd[p], i);
            eh = lds_read_b128(ehi_at + (unsigned)(p * kHiRows * HROW * 16));
            // the next slice sets out spread over this one's rounds; its phase factors and queries in the last round
            if (more) {
                if (TWO && p == 0 && i < SETS) send_set(sl + 1, i);
                if (p == (NP - 1) / 2 && i == PL - 1) aux_load(sl + 1);
            }
            // (cleared by a small matrix instruction: the compiler makes five moves of a vector of zeros)
            acc = __builtin_amdgcn_mfma_f32_4x4x1f32(zero, zero, floatx4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
            for (int st = 0; st < NST; ++st) {
                const uint4_t pa = v[(p * NST + st) % NBUF][0], pb2 = v[(p * NST + st) % NBUF][1];
                const uint8v_t both = {pa[0], pa[1], pa[2], pa[3], pb2[0], pb2[1], pb2[2], pb2[3]};
                acc = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(selv, __builtin_bit_cast(bf16x16_t, both), acc, (int)sidx, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (st + NBUF < NST) issue(p, st + NBUF);
                else if (p + 1 < NP) issue(p + 1 < NP ? p + 1 : p, st + NBUF - NST);
                __builtin_amdgcn_sched_barrier(0);
                part(st);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        auto pair = [&](auto kc) __attribute__((always_inline)) {
            constexpr int k = decltype(kc)::value;
            pass(std::integral_constant<int, 2 * k>{}, acc_e, eh_e, [](int) {});
            if (k == 0 || (chg >> (2 * k - 1) & 7u)) fold(k);
            if constexpr (2 * k + 1 < NP) {
                pass(std::integral_constant<int, 2 * k + 1>{}, acc_o, eh_o, [&](int st) { if (st < 2) rotate(st, acc_e, eh_e, xy); });
            } else {
                rotate(0, acc_e, eh_e, xy);
                rotate(1, acc_e, eh_e, xy);
                acc_o = floatx4_t{0.f, 0.f, 0.f, 0.f};
                eh_o = uint4_t{0u, 0u, 0u, 0u};
            }
#pragma unroll
            for (int st = 0; st < NST; ++st) finish(k, st);
        };
        // (even and odd passes' sums and factors in turn)
        auto half = [&](auto pc) __attribute__((always_inline)) {
            constexpr int p = decltype(pc)::value;
            if constexpr (p < NP) {
                typedef std::integral_constant<int, (p > 0 ? p - 1 : 0)> before;
                if constexpr (p % 2 == 0) pass(pc, acc_e, eh_e, [&](int st) { if (p > 0) finish_half(before{}, acc_o, eh_o, st); });
                else pass(pc, acc_o, eh_o, [&](int st) { finish_half(before{}, acc_e, eh_e, st); });
                if (p == 0 || (chg >> p & 1u)) fold(p);
                if constexpr (p == NP - 1) {
#pragma unroll
                    for (int st = 0; st < NST; ++st) finish_half(pc, p % 2 ? acc_o : acc_e, p % 2 ? eh_o : eh_e, st);
                }
            }
        };
#pragma unroll
        for (int st = 0; st < NBUF; ++st) issue(0, st);
        if constexpr (HALF) {
            half(std::integral_constant<int, 0>());
            half(std::integral_constant<int, 1>());
            half(std::integral_constant<int, 2>());
            half(std::integral_constant<int, 3>());
            half(std::integral_constant<int, 4>());
            half(std::integral_constant<int, 5>());
            half(std::integral_constant<int, 6>());
            half(std::integral_constant<int, 7>());
        } else {
            pair(std::integral_constant<int, 0>());
            if constexpr (NPAIR > 1) pair(std::integral_constant<int, (NPAIR > 1 ? 1 : 0)>());
            if constexpr (NPAIR > 2) pair(std::integral_constant<int, (NPAIR > 2 ? 2 : 0)>());
            if constexpr (NPAIR > 3) pair(std::integral_constant<int, (NPAIR > 3 ? 3 : 0)>());
        }
    }
    }

    // Write-out.  A wavefront's tokens are scattered over the pass (4 fine positions x 8 coarse rows), so the logits of
    // four heads at a time are transposed through the now idle codebook blocks, [head][pass][coarse row][68] floats (rows
    // padded from 64: the 64 lanes of a write fall on 64 different banks), and leave as runs of 256 consecutive tokens
    // per wavefront, whose (max, sum of exp) are taken on the way.  A slice group leaves partial logits in its own array;
    // the statistics then come from k_score_combine.
    float *stg = reinterpret_cast<float *>(tab);
    float2 *wst = reinterpret_cast<float2 *>(reinterpret_cast<char *>(tab) + WST_AT);
    const int4 *segs = reinterpret_cast<const int4 *>(reinterpret_cast<const char *>(tab) + SEG_AT);
    float *dst0 = scores + (size_t)eg * a.part_stride;
    const int ln = fresh_lane(), wpar = ln >> 4 & 1, wf = 4 * wave + (ln >> 2 & 3), wrow = (ln & 3) + 4 * (ln >> 5);
    const int wp = wave >> 1, rel = ((wave & 1) * 64 + ln) * 4;  // the pass and the 4 tokens this thread writes
#pragma unroll
    for (int x = 0; x < NGRP; ++x) {
        __syncthreads();  // the last slice (x = 0) or the previous group's logits have been read by everyone
#pragma unroll
        for (int k = 0; k < NPAIR; ++k)
            if (2 * k < np) {
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    const float v = HALF ? swap16_add(sc[2 * k % NV][x][h], 2 * k + 1 < NP ? sc[(2 * k + 1) % NV][x][h] : 0.f) : sc[k][x][h];
                    if (2 * k + wpar < NP) stg[((h * NP + 2 * k + wpar) * 8 + wrow) * 68 + wf] = v * a.scale;
                }
            }
        __syncthreads();
        if (wp < np) {
            const int4 sg = segs[wp];
            const int L = __builtin_amdgcn_readfirstlane(sg.z), t0 = __builtin_amdgcn_readfirstlane(sg.y);
            const int c0 = __builtin_amdgcn_readfirstlane(sg.w);
            const int tok = t0 + rel;
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                if (4 * x + h >= G) break;
                const float4 w = *reinterpret_cast<const float4 *>(stg + ((h * NP + wp) * 8 + (rel >> kLoBits)) * 68 + (rel & (kLo - 1)));
                const __amdgpu_buffer_rsrc_t row = make_rsrc(dst0 + (size_t)c0 * a.Hq + (size_t)(g * G + 4 * x + h) * L, (unsigned)L * 4u);
                if (tok + 3 < L) {                            // (rows begin at any multiple of 4 bytes)
                    store_through(__builtin_bit_cast(uint4_t, w), row, (unsigned)tok * 4u);
                } else {
                    if (tok < L) store_through(w.x, row, (unsigned)tok * 4u);
                    if (tok + 1 < L) store_through(w.y, row, (unsigned)tok * 4u + 4u);
                    if (tok + 2 < L) store_through(w.z, row, (unsigned)tok * 4u + 8u);
                }
                if (a.groups == 1) {
                    const float w0 = tok < L ? w.x : -INFINITY, w1 = tok + 1 < L ? w.y : -INFINITY;
                    const float w2 = tok + 2 < L ? w.z : -INFINITY, w3 = tok + 3 < L ? w.w : -INFINITY;
                    const float m = wave_max(fmaxf(fmaxf(w0, w1), fmaxf(w2, w3)));
                    float l = 0.f;
                    if (m != -INFINITY)
                        l = __builtin_amdgcn_exp2f((w0 - m) * kLog2e) + __builtin_amdgcn_exp2f((w1 - m) * kLog2e) +
                            __builtin_amdgcn_exp2f((w2 - m) * kLog2e) + __builtin_amdgcn_exp2f((w3 - m) * kLog2e);
                    l = wave_sum(l);
                    if (ln == 0) wst[wave * 8 + 4 * x + h] = make_float2(m, l);
                }
            }
        }
    }
    if (a.groups == 1) {
        __syncthreads();
        const int x = wave * 64 + ln;
        if (x < np * G) {
            const int p = x / G, h = x % G;
            const int4 sg = segs[p];
            const float2 s0 = wst[2 * p * 8 + h], s1 = wst[(2 * p + 1) * 8 + h];  // (the first half is never empty)
            float l = s0.y;
            const float m = fmaxf(s0.x, s1.x);
            l *= __builtin_amdgcn_exp2f((s0.x - m) * kLog2e);
            if (s1.x != -INFINITY) l += s1.y * __builtin_amdgcn_exp2f((s1.x - m) * kLog2e);
            sstat[((size_t)sg.x * a.Hq + (size_t)g * G + h) * a.nstat + sg.y / kPassTokens] = make_float2(m, l);
        }
    }
}


}  // namespace
