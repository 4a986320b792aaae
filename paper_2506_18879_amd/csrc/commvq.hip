// libcommvq: decode attention over a CommVQ-compressed KV cache, hand-written for gfx950.
//
// Pipeline of one call (all on the caller's stream):
//   score stage Eq. new_attention: per (token, KV head) gather-sum the M_k selected key
//               codewords, rotate once by the RoPE matrix of the relative position, contract
//               with the G query heads of the group -> scaled logits + per-split (max, sum exp).
//               bf16 codebooks with contiguous key positions: k_prep (codebook re-laid in
//               LDS-image order) + k_score_stream (codebook slices streamed through LDS, tile codes
//               resident in registers, gather-sum and query contraction on the matrix cores), for
//               short contexts with the tiles also cut along the slices + k_score_combine;
//               fp32 codebooks, explicit key positions: k_score (rows gathered through L1); those and other keys in launches of few
//               tokens: k_score_few.
//   k_values    Softmax(A) S_V of Eq. optimized_v and its product with the value codebook (commvq_values.hpp): exp(logit - max) is
//               scatter-added into LDS bins, one per head, value codebook and codeword, in 32-bit fixed point (integer LDS
//               atomics run ~20x faster than fp32 ones on gfx950), and the bins are multiplied by the codebook rows on the matrix
//               cores.  Binary value code: k_vbits, then k_out or k_out_mfma with the bins in memory in between.
//   k_out_final sum of the partial products, division by the softmax denominator.
// Key encoding for cache append lives in commvq_encode.hip, the EM codebook learner in commvq_em.hip.
//
// RoPE algebra used by k_score (Sec. 3.2, Eq. rope_ri).  Writing a 2-D sub-vector (x, y) as
// z = x + iy, the paper's row-vector product (x, y) R_m^j is z * exp(-i m theta_j).  The dot
// product of two sub-vectors is Re(a conj(b)), so
//     (q^j R_t^j) . (k^j R_p^j) = Re( q^j conj(k^j) exp(-i (t - p) theta_j) ),
// i.e. only the relative position t - p enters, and the rotation can be applied to the
// gather-summed codewords once per token (commutativity, Property 1).
#include <algorithm>
#include <cstring>

#include "commvq_internal.hpp"
#include "commvq_values.hpp"
#include "commvq_vbits.hpp"

// Scratch memory of commvq_decode_attn_static: the workspace of a call, held by the library itself so that the
// entry point allocates nothing.  One copy per GPU the library is loaded on, for the life of the process.  In host
// code this name is only a stand-in for the symbol: the device address is looked up once per device in
// commvq_create (hipGetSymbolAddress) and kept in the handle; kernels receive that pointer.
constexpr size_t kStaticScratchBytes = (size_t)48 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

struct Workspace {
    float2 *sstat;    // [B * Hq * score_splits] (max, sum of exp(logit - max)) of each score split
    float *scores;    // [T * Hq] scaled logits
    // written and read by the value and output stages only
    float *vscale;    // [B * Hq * value_splits] 2^-S: value of one fixed-point unit of that split's bins
    float *lsum;      // [B * Hq * value_splits] sum of exp(logit - sequence max) over the score tiles that begin in that value split
    unsigned *bins;   // [B * Hkv * value_splits][K][Mv][G] fixed-point bins (binary values; stage calls of indexed ones)
    float *partial;   // [B * Hq * out_chunks][d]
    uint4 *packed_val;    // value codebook re-laid for k_out_mfma (batches; only if the caller has not packed it)
    // written and read by the score stage only, in the same memory as the above; in front of them, right behind `scores`, the
    // partial logits of slice groups 1, 2, .. when the score tiles are also cut along the slices (group 0's are in `scores`)
    uint4 *packed;    // key codebook re-laid slice-major for k_score_stream / k_score_pair
    float *lut;           // position-free keys: scale * q . C, [B * Hkv][M_k * K][G]
    size_t bytes;
};

// The slice-streaming score kernel (k_score_stream) serves bf16 codebooks with contiguous positions; everything else
// (fp32 codebooks, explicit key positions) goes through the gather kernel.
bool use_sliced(const commvq_handle *h, bool explicit_positions)
{
    if (h->cfg.position_free) return true;  // scalar look-up table kernel: same tiling, positions play no role
    return h->cfg.codebook_dtype == COMMVQ_BF16 && !explicit_positions;
}

// The batched output kernel (value codebook on the matrix cores) serves bf16 codebooks from 16 output rows
// (sequences x query heads of a KV head) on.
inline bool use_out_mfma(const commvq_handle *h, int batch)
{
    return h->cfg.codebook_dtype == COMMVQ_BF16 && batch * h->G >= kOutMfmaMinRows;
}

// Binary value code: N_c code bits per token for all KV heads, one codebook [N_c][Hkv * d].  Towards the output kernels a
// KV head's N_c bins stand in for N_c / 256 value codebooks of 256 rows; bins row r is code bit vbits_code_bit(r).
inline bool bin_values(const commvq_config &c) { return c.value_format == COMMVQ_VALUES_BINARY; }
inline int val_books(const commvq_config &c) { return bin_values(c) ? c.value_bits / kK : c.m_val; }

// Paired-code key format: blocks of 16 levels (sizes), bytes of one packed record.
inline bool pair_keys(const commvq_config &c) { return c.key_format == COMMVQ_KEYS_PAIRED; }
inline int pair_blocks(const commvq_config &c) { return (c.key_levels + 15) / 16; }
inline int pair_record_bytes(const commvq_config &c) { return (12 * c.key_levels + 7) / 8; }
// Sets of four levels that the kernels work on: levels beyond key_levels are zeros (R = 11: 3 sets, R = 21: 6).
inline int pair_sets(const commvq_config &c) { return c.key_levels <= 12 ? 3 : c.key_levels <= 16 ? 4 : 6; }
constexpr int kPairSlices = 4;  // LDS slices of four planes
// Passes of k_score_pair at most (2, 3, 4 or these).
constexpr int pair_passes(int sets) { return sets == 3 ? 8 : 6; }
// Memory that paired keys have had in a workspace beside the packed table (an index byte per level, unpacked): partial logits may use it.
inline size_t pair_room(const commvq_config &c, int64_t T) { return pair_keys(c) ? (size_t)T * c.n_kv_heads * 32 * pair_blocks(c) : 0; }
inline size_t packed_key_bytes(const commvq_config &c)
{
    if (pair_keys(c)) return (size_t)c.n_kv_heads * 16 * pair_blocks(c) * 64 * 256;  // 16 planes x blocks x 16 KiB
    return (size_t)c.n_kv_heads * c.m_key * kK * kD * 2;
}

// Value split for score tiles of slen tokens (1024 where k_score_combine writes the statistics).
int value_split_len(const commvq_handle *h, int B, int max_seqlen, int slen)
{
    const int units = B * h->cfg.n_kv_heads;
    int nv = 256 / units;  // about one value workgroup per compute unit
    if (bin_values(h->cfg))  // a workgroup of the binary-code value kernel: 16 query heads x 1024 code bits of one token range
        nv = 256 / (B * ((h->cfg.n_q_heads + kVbitsHeads - 1) / kVbitsHeads) * (h->cfg.value_bits / kVbitsCols));
    if (nv < 1) nv = 1;
    int vlen = (max_seqlen + nv - 1) / nv;
    // a whole number of tiles, or a power-of-two fraction of one (never less than 1024 tokens): k_vbits takes its exp-sums from
    // the tiles' statistics.  (k_score_stream's are per 512 tokens, so there the tile is more than would be necessary.)
    if (vlen >= slen || slen <= 1024) {
        const int round_to = slen > 1024 ? slen : 1024;
        vlen = (vlen + round_to - 1) / round_to * round_to;
    } else {
        int part = 1024;
        while (part < vlen) part *= 2;
        vlen = part;  // 1024 or 2048 inside a 2048- or 4096-token tile
    }
    // the binary-code value kernel sums signed digit x bit products in 32-bit accumulators: |digit| <= 2^7, |bit byte| <= 2^7,
    // so a range of at most 2^16 tokens stays within 2^30
    if (bin_values(h->cfg) && vlen > (1 << 16)) vlen = 1 << 16;
    return vlen;
}

// Bytes of the logits, and from one slice group's partial logits to the next's.
inline size_t logit_bytes(const commvq_handle *h, int64_t T) { return align_up((size_t)T * h->cfg.n_q_heads * 4, 256); }

// Partial output rows per head in the workspace, and whether it has a place for the packed value codebook.  Indexed values need neither
// so many rows nor the codebook: their batches' workspaces keep the sizes they have had.  With paired keys the statistics, one per
// 512 tokens, take some of it instead (batches: 256 codebook rows per partial row).
inline size_t partial_rows(const commvq_handle *h, int B)
{
    const size_t rows = (size_t)val_books(h->cfg) * kK;
    return pair_keys(h->cfg) && use_out_mfma(h, B) ? rows / kOutMfmaRows : rows / kOutRows;
}
inline bool packed_value_room(const commvq_handle *h, int B) { return use_out_mfma(h, B) && (bin_values(h->cfg) || !pair_keys(h->cfg)); }

// Bytes of the workspace that only the value and output stages use (Workspace: vscale to packed_val).
size_t value_stage_bytes(const commvq_handle *h, int B, size_t vsplits)
{
    const commvq_config &c = h->cfg;
    const size_t rows = (size_t)val_books(c) * kK, heads = (size_t)B * c.n_q_heads;
    return 2 * align_up(heads * vsplits * 4, 256) + align_up(heads * vsplits * rows * 4, 256) + align_up(heads * partial_rows(h, B) * kD * 4, 256) +
           (packed_value_room(h, B) ? align_up((size_t)c.n_kv_heads * rows * kD * 2, 256) : 0);
}

// Launches of so few tokens that 1024-token tiles leave compute units without one: a tile's partial logits for each unit.
size_t few_tile_bytes(const commvq_handle *h, int B, int64_t T, int max_seqlen)
{
    if (pair_keys(h->cfg)) return 0;
    const int64_t tiles = (int64_t)B * h->cfg.n_kv_heads * ((max_seqlen + 1023) / 1024);
    int64_t cut = 1;
    while (2 * cut <= h->cfg.m_key / 2 && 2 * cut * tiles <= 256) cut *= 2;
    return cut > 1 ? (size_t)cut * logit_bytes(h, T) : 0;
}

// Where the value stage's arrays begin (carve): `shared` is the end of the partial logits, `parts` their size, `packed` what the score stage
// has behind them.
inline size_t value_stage_at(size_t shared, size_t parts, size_t packed, size_t few, size_t value)
{
    const size_t apart = few ? few + std::min(packed, value) : 0;
    return shared - (parts > apart ? parts - apart : 0);
}

// Tokens of a workgroup of the row-gather kernels.
int gather_split_len(int units, int max_seqlen)
{
    int len = 1024;
    // down to 4 tokens per wavefront (one iteration of four tokens): a short context still spreads over the chip
    while (len > kFewTokens && (long)units * ((max_seqlen + len - 1) / len) < kScoreMinWgs) len /= 2;
    return len;
}

// How k_score_stream cuts a launch: `passes` segments of 512 tokens per workgroup, `tiles` workgroups per KV head, each of
// them once per slice group.
struct StreamShape {
    int passes, tiles, groups;
};
// Cost of a workgroup in microseconds: a fixed start and end (launch, first fetches, write-out), and per slice a switch and the
// passes.  A launch too short to fill the 256 compute units is also cut along the slices; every group then fetches the tile's codes
// again, the partial logits take a trip through memory, and k_score_combine is one more launch.
struct StreamCost {
    double fixed, change, pass, combine, group, logits;  // (the last two per slice group; logits per million)
};
StreamShape stream_shape(const commvq_handle *h, int B, int64_t T, int max_seqlen)
{
    const int per_seq = (max_seqlen + kPassTokens - 1) / kPassTokens;
    // segments per KV head: at most one partly filled one per sequence more than the tokens need
    const int64_t most = std::min<int64_t>((int64_t)B * per_seq, T / kPassTokens + B);
    const bool pair = pair_keys(h->cfg);
    const int sets = pair_sets(h->cfg);
    // What the host does not know is how many of them are partly filled: half of the sequences' last ones on average, with a standard deviation
    // of sqrt(B / 12).  k_score_stream: a cut is judged by that mean and by one deviation to either side of it, since one segment more than fills
    // the compute units is a second round (8 sequences of 2000 to 4000 tokens, 32 codebooks 50.6 -> 34.8 us, 64 of 1500 to 3000 154.5 -> 141.6
    // with the mean alone and so).  k_score_pair: by a whole number of deviations more than the mean (8 sequences of 1250 to 2500 tokens 71.3 us
    // by the mean, 63.2 so).
    int spread = 0;
    while (pair && B > 1 && 12 * spread * spread < B) ++spread;
    // (k_score_stream: no fewer than the sequences, or a batch of short ones is taken for half of what it is.  Whole calls in microseconds, 64
    // sequences of up to 233 tokens, 8 x 8 heads, 32 codebooks 120.8 -> 95.3; 2 x 8 heads, 64 of up to 116 48.2 -> 37.4; 8 x 4 heads, 57 of up to 307
    // 101.9 -> 85.6, with 16 codebooks 50 of up to 270 66.2 -> 55.0.)
    const bool known = B == 1 || per_seq == 1 || T == (int64_t)B * max_seqlen;
    const double mean = known ? (double)B * per_seq : (double)T / kPassTokens + 0.5 * B, dev = known ? 0.0 : std::sqrt(B / 12.0);
    auto segments = [&](int k) -> int64_t {                   // k = -1, 0, 1
        if (pair) return B == 1 ? most : std::min<int64_t>((int64_t)B * per_seq, T / kPassTokens + (B + 1) / 2 + spread);
        return std::max<int64_t>(B, std::min<int64_t>((int64_t)B * per_seq, (int64_t)(mean + k * dev + 0.5)));
    };
    // k_score_stream, fitted to every cut (2 to 8 passes, 1 to 16 groups) of 28 shapes of 2900 to 131072 tokens and 1 to 64 sequences; the cut
    // chosen is 0.3 % slower than the best on average.  One sequence of at most 32 segments keeps the numbers of an older form of
    // the kernel, for the sake of the cut that a test names at 16384 tokens and not of its speed (1 to 6 % slower than the best).
    // (One sequence of 32768 tokens, 32 codebooks 38.9 -> 36.7 us; 24 of 300 to 600 45.7 -> 29.2; 40 of 1500 to 3000 92.6 -> 83.9.)
    const bool two = h->cfg.m_key == 32, wide = h->G == 8;
    const StreamCost cost = B == 1 && most <= 32
        ? StreamCost{9.0, two ? 1.25 : wide ? 0.6 : 0.5, two ? (wide ? 0.70 : 0.66) : (wide ? 0.47 : 0.41), 5.0, two ? 0.08 : 0.15, 1.0}
        : two ? (wide ? StreamCost{3.18, 1.40, 0.687, 3.04, 0.355, 1.23} : StreamCost{2.57, 1.03, 0.584, 2.06, 0.375, 2.39})
              : (wide ? StreamCost{1.70, 0.917, 0.483, 2.73, 0.855, 1.51} : StreamCost{2.35, 0.747, 0.352, 2.63, 0.715, 1.49});
    // Launches of at most 64 segments x KV heads: one more slice group costs little there.  Fitted to every cut of 112 batches of 100 to 80000
    // tokens, 1 to 64 sequences, 1 to 16 KV heads: the cut chosen is 0.5 % slower than the best on average, 2.9 % with the costs above for
    // all (KV heads x query heads each, microseconds: 1 x 4, 3 sequences of up to 1025 tokens, 16 codebooks 23.5 -> 18.9; 2 x 4, 8 of up to 139, 32
    // codebooks 21.5 -> 19.4; 1 x 8, 5 of up to 876 24.4 -> 22.0); with the line at 256 some of those beyond it are 3 to 5 % slower.
    const double group = segments(0) * h->cfg.n_kv_heads <= 64 && !(B == 1 && most <= 32) ? (two ? 0.2 : 0.15) : cost.group;
    // k_score_pair: 16 rounds, four to a slice; 2, 3, 4 or pair_passes passes.  Fitted to 29 shapes of 2000 to 131072 tokens, 1 to 8
    // sequences, R = 11 and 21: 15 cuts each, the one chosen is 0.7 % slower than the best on average (8 sequences of 1100 to 2200 tokens, R = 11:
    // 55.9 us with groups of 8 rounds, 63.0 uncut; one of 2000: 39.9 with groups of two rounds, 56.8 uncut).
    // Three passes where two do not fit one workgroup per compute unit and four leave too many of them idle, best of the others -> three:
    // R = 21, one sequence of 17000 tokens 70.7 -> 65.2 us, of 9000 56.3 -> 53.1; R = 11, 40000 tokens 75.1 -> 70.8, 16 sequences of 1500 to
    // 3000 85.3 -> 80.7.  Uncut with six sets of levels it loses to six passes in two groups (two sequences of 10000 to 20000: 90.2 against 94.3).
    // Two passes of three sets uncut take 2.5 us (8 heads per KV head: 5) more than the line through the others (their rounds are too short
    // for the codes on their way): 8 sequences of 1374 to 2748 tokens 64.7 us, 63.2 with three passes in two groups; 8 heads, one of 17000 63.5 and 61.3.
    const double pc = (wide ? 0.10 : 0.0) + (sets == 3 ? 0.443 : sets == 4 ? 0.535 : 0.728);
    // The partial logits may not need more memory than the bins that follow them, apart from few_tile_bytes: a shape that fits a
    // workspace of some size (the static one in particular) must not outgrow it for the sake of a faster cut.
    const int vlen = value_split_len(h, B, max_seqlen, 1024);
    const size_t one = logit_bytes(h, T);
    const size_t value = value_stage_bytes(h, B, (size_t)(max_seqlen + vlen - 1) / vlen);
    const size_t few = few_tile_bytes(h, B, T, max_seqlen);
    size_t room = value + few;
    if (pair) {  // no more than the shape has needed with unpacked indices, or 32 MB in all
        const size_t rest = one + packed_key_bytes(h->cfg) + align_up((size_t)B * h->cfg.n_q_heads * per_seq * 8, 256), small = (size_t)32 << 20;
        room = std::max({pair_room(h->cfg, T), value - std::min(value, packed_key_bytes(h->cfg)), small - std::min(small, rest)});
    }
    // Nor may a shape outgrow the static array that fits it uncut (behind the partial logits lies the re-laid codebook, too: 40 sequences of up
    // to 29503 tokens, 707107 in all, one query head each: 47 MB uncut, 62 in two groups).
    const int gather = gather_split_len(B * h->cfg.n_kv_heads, max_seqlen);
    const size_t stats = align_up((size_t)B * h->cfg.n_q_heads * std::max(per_seq, (max_seqlen + gather - 1) / gather) * 8, 256);
    auto bytes = [&](size_t parts) {
        const size_t shared = stats + one + parts, packed = packed_key_bytes(h->cfg);
        return std::max(shared + packed, value_stage_at(shared, parts, packed, few, value) + value);
    };
    const size_t most_bytes = bytes(0) <= kStaticScratchBytes ? kStaticScratchBytes : SIZE_MAX;
    StreamShape best = {2, 1, 1};
    double t_best = 1e30;
    const double million = (double)T * h->cfg.n_q_heads / 1e6;  // logits
    const int most_passes = pair ? pair_passes(sets) : kStreamPasses;
    for (int passes = 2; passes <= most_passes; passes = !pair || passes != 4 ? passes + 1 : most_passes)
        for (int e = 1; e <= kStreamSlices && (e - 1) * one <= room; e *= 2) {
            if (pair && passes == 3 && e == 1 && sets > 3) continue;
            if (!pair && bytes((e - 1) * one) > most_bytes) continue;
            const double slices = (double)kStreamSlices / e;
            auto rounds = [&](int64_t segs) { return (double)(((segs + passes - 1) / passes * h->cfg.n_kv_heads * e + 255) / 256); };
            double t;
            if (pair) {
                t = rounds(segments(0)) * (9.4 + std::max(1.0, slices / 4) * 0.32 + slices * (0.27 + passes * pc)) +
                    (e > 1 ? 4.8 + e * 3.35 * million : passes == 2 && sets == 3 ? (wide ? 5.0 : 2.5) : 0.0);
            } else {
                const double n = dev > 0.0 ? 0.3 * rounds(segments(-1)) + 0.4 * rounds(segments(0)) + 0.3 * rounds(segments(1)) : rounds(segments(0));
                t = n * (cost.fixed + slices * (cost.change + passes * cost.pass)) + (e > 1 ? cost.combine + e * (group + cost.logits * million) : 0.0);
            }
            if (t < t_best * 0.9999) { t_best = t; best = StreamShape{passes, 0, e}; }
        }
    best.tiles = (int)((most + best.passes - 1) / best.passes);
    return best;
}

// Whether the sliced score path is k_score_stream or k_score_pair (keys with RoPE), not the look-up table.
inline bool stream_keys(const commvq_config &c) { return !c.position_free; }

// Whether up to 4 heads take k_score_stream's and k_score_pair's exchange of rows within a pair of passes, as 8 heads do, and not logits in
// halves.  Halves save the exchange but fold the queries in every pass that begins another sequence where an exchanged pair does so
// once, and a launch of one round is as slow as its slowest workgroup.  They lose for a batch with two passes a workgroup, and with an even number
// of passes where most of them are a sequence of its own.  Whole calls in microseconds, halves and exchange: two passes, 24 sequences
// of 750 to 1500 tokens, 16 codebooks 48.8 and 47.7, R = 11 54.2 and 52.3, 8 of 1750 to 3500 43.5 and 42.3, 49.2 and 46.9 (one sequence of 30000: 37.7 and
// 39.4, 42.2 and 43.8); four passes, 64 of 280 to 560 71.2 and 68.7, 85.4 and 81.8 (40 of 550 to 1100: 65.4 and 65.9, 78.4 and 78.0; 16 of 2048 to 4096: 54.5
// and 57.4, 66.2 and 68.9).  Exchange against halves over every cut of 180 batches, on average: two passes in slice groups 0.98 to 0.99; short
// sequences with four, six and eight 0.97 to 0.98, with an odd number 0.99 to 1.03; long ones with four and more 1.00 to 1.02.  32
// codebooks: no more than 0.9 us either way with short sequences, else halves by 1 to 12.  (The exchange adds a token's 8 products in one chain,
// halves in two of 4: rms error of the logits 1.25e-7 and 1.06e-7.)
inline bool exchange_rows(const commvq_handle *h, const StreamShape &s, int B, int64_t T)
{
    if (h->G == 8 || B == 1 || (!pair_keys(h->cfg) && h->cfg.m_key == 32)) return false;
    return s.passes == 2 || (s.passes % 2 == 0 && T <= (int64_t)B * kPassTokens);
}

// Whether gathering rows (k_score_few) serves a launch of bf16 codebooks with contiguous positions better than the slices: so few
// tokens that 16 of them a workgroup leave none of it waiting and the rows' way through the L1s (tokens x heads x codebooks x 256
// bytes) costs less than the partial logits and their sum.  Whole calls, slices -> rows, in microseconds, 8 KV heads: 4 query heads each and 16 +
// 16 codebooks 200 tokens 18.3 -> 14.4, 1237 21.5 -> 14.9, 4000 24.2 -> 20.6, 6000 27.3 -> 24.6, 8000 27.3 -> 28.4; 32 + 32 codebooks 200
// tokens 18.5 -> 13.6, 1237 24.7 -> 19.6, 2500 26.9 -> 23.6, 3200 27.0 -> 26.9, 4000 27.4 -> 28.8; 8 query heads each and 32 + 32 codebooks
// 1237 tokens 27.9 -> 22.8, 2500 30.8 -> 27.2, 3200 30.0 -> 31.4; 24 sequences of 256, 16 + 16 codebooks 35.3 -> 29.1; 32 KV heads of 4,
// 32 + 32 codebooks 300 tokens 34.2 -> 27.9, 1000 36.6 -> 42.1.  Layers of fewer than 8 KV heads keep the slices, not
// because they are faster there (two KV heads of 4, 16 + 16 codebooks: 1500 tokens 20.8 us, with rows 17.4, 6000 20.8 and 17.0) but because the tests of
// the slices are written for such layers.
inline bool few_tokens(const commvq_handle *h, int B, int64_t T, int max_seqlen)
{
    const commvq_config &c = h->cfg;
    return !pair_keys(c) && c.n_kv_heads >= 8 && T * c.n_kv_heads * c.m_key <= 700000 &&
           (int64_t)B * c.n_kv_heads * ((max_seqlen + 2 * kFewTokens - 1) / (2 * kFewTokens)) < kScoreMinWgs;
}

// Indexed values go through k_values, the binary code through k_vbits and the output kernels.
inline bool fused_values(const commvq_config &c) { return !bin_values(c); }

// How k_values cuts a launch: codebooks per workgroup, whole sequences per workgroup (1: a token range of one), column
// parts, threads, token ranges per sequence and their length, tokens of a range that share a fixed-point unit.
struct ValueShape {
    int books, slots, parts, threads, ranges, range_len, span;
};

// A plan and what of the kernels' shapes the public part does not say.
struct Plan : commvq_plan {
    StreamShape stream;
    ValueShape values;
};

// Granularity of the (max, sum of exp) statistics that the score stage leaves for the value stage: the score tile, except that
// k_score_stream writes them per 512-token segment and k_score_combine (tiles cut along the slices) per 1024 tokens.
inline int stat_len(const commvq_handle *h, const Plan &p)
{
    if (p.score_kernel && stream_keys(h->cfg)) return p.score_slice_groups > 1 ? 1024 : kPassTokens;
    return p.score_split_len;
}
inline int stat_splits(const commvq_handle *h, const Plan &p, int max_seqlen) { return (max_seqlen + stat_len(h, p) - 1) / stat_len(h, p); }

// splits, split_len: value splits per sequence that the workspace holds, and their length; tile: tokens of a statistics tile.
// Spans are two value splits long (k_values), ranges whole tiles: a tile that two spans share counts towards both their units, and
// those may be no coarser than what a value split or a tile gives.  Whole calls in microseconds, one choice against the other:
//  * 4 codebooks a workgroup, so that a token range is long where a sequence has few heads: 9001 tokens 36.3 against 38.4
//    with 8, 1237 tokens 24.7 against 26.4; from 128 groups of four on (64 of 8 heads) 8, which compute half as many
//    exponentials: 8 x 8K..64K 456 against 499, 4 x 2.5K..20K (at the line) 56.6 against 55.0;
//  * 1024 threads, one workgroup per compute unit, which then reads its codebook rows once: 9001 tokens 36.3 against 39.1
//    with 512, 60001 tokens 53.4 against 57.5; where there are more workgroups than compute units anyway two of 512 run
//    side by side: 40 x 1500..3000 105.9 against 110.2, 12 x 1K..9K of 8 heads 114.3 against 116.3;
//  * whole sequences side by side, four of 4 heads or two of 8 (128 KiB of bins), which share the codebook rows, once that leaves
//    256 workgroups and the sequences are short: 64 x 512..1024 119.7 against 132.2 one by one, 30 x 300..600 of 8 heads
//    83.1 against 89.9; with ranges of 2250 tokens on average no gain (107.4 against 105.9);
//  * a quarter of the columns each where not even 64 workgroups would be there: 300 tokens 17.6 against 19.5, 2000 tokens
//    20.7 against 22.2 (with 64: 24.7 either way; with 256: 61 against 79).
ValueShape value_shape(const commvq_handle *h, int B, int64_t T, int max_seqlen, int splits, int split_len, int tile)
{
    const int G = h->G, M = h->cfg.m_val, units = B * h->cfg.n_kv_heads;
    const bool wide = h->cfg.codebook_dtype == COMMVQ_BF16 && G >= 4;
    ValueShape v = {4, 1, 1, wide ? 1024 : 512, 1, 0, 2 * std::max(split_len, tile)};
    if (wide && (int64_t)G * units * M > 2048) {
        v.books = 8;
        const int groups = units * (M / 8);
        if (T <= (int64_t)B * 1536) {
            if (G == 4 && groups >= 1024) v.slots = 4;
            else if (groups >= 512) v.slots = 2;
        }
        if (groups > 256) v.threads = 512;
    }
    const int groups = units * (M / v.books);
    // as many ranges as there is place for bins (stage by stage) and output rows
    int n = std::max(1, (v.threads == 512 ? 512 : 256) / groups);
    // (two workgroups on a compute unit have no LDS for the sums of several spans: at most two ranges, since a sequence then has three splits at most)
    if (wide && v.threads == 512) n = std::max(n, (max_seqlen + v.span - 1) / v.span);
    n = v.slots > 1 ? 1 : std::max(1, std::min(n, std::min(splits, (int)partial_rows(h, B) * v.books / M)));
    const int step = std::max(512, tile);
    v.range_len = std::max(1024, ((max_seqlen + n - 1) / n + step - 1) / step * step);
    v.ranges = v.slots > 1 ? 1 : (max_seqlen + v.range_len - 1) / v.range_len;
    if (v.slots > 1) v.range_len = v.span = max_seqlen;  // (128 of these at least: two value splits at most)
    v.span = std::min(v.span, v.range_len);
    if (v.books == 4 && (int64_t)groups * v.ranges * 4 <= 256) v.parts = 4;
    return v;
}

void make_plan(const commvq_handle *h, int B, int64_t T, int max_seqlen, bool sliced, Plan *p)
{
    const int units = B * h->cfg.n_kv_heads;
    int len;
    p->stream = StreamShape{0, 0, 1};
    if (sliced && stream_keys(h->cfg) && few_tokens(h, B, T, max_seqlen)) sliced = false;
    if (sliced && stream_keys(h->cfg)) {
        p->stream = stream_shape(h, B, T, max_seqlen);
        len = 1024;  // what is reported, and value splits are cut by: the workgroup's tokens rounded up to a power of two
        while (len < p->stream.passes * kPassTokens) len *= 2;
    } else if (sliced) {
        // Tile = 1024, 2048 or 4096 tokens of one (sequence, KV head).  Cost model of a workgroup, in microseconds: a fixed
        // start (first fetches, write-out), per slice a switch (LDS refill, barriers) and the passes themselves.
        const int S = h->cfg.m_key / 2;                       // slices per tile
        const double c1024 = h->cfg.m_key == 16 ? 2.1 : 1.85;  // passes of 1024 tokens over one slice
        double best = 1e30;
        len = 1024;
        for (int tpt = 1; tpt <= kScoreMaxTpt; tpt *= 2) {
            if (tpt == 4 && h->G == 8 && h->cfg.m_key == 16) break;  // those instantiations run out of registers
            const long wgs = (long)units * ((max_seqlen + 1024 * tpt - 1) / (1024 * tpt));
            const double t = (double)((wgs + 255) / 256) * (9.0 + (double)S * (1.3 + tpt * c1024));
            if (t < best * 0.9999) { best = t; len = 1024 * tpt; }
        }
    } else {
        len = gather_split_len(units, max_seqlen);
    }
    const int groups = p->stream.groups;
    p->score_split_len = len;
    p->score_splits = (max_seqlen + len - 1) / len;
    const int vlen = value_split_len(h, B, max_seqlen, groups > 1 ? 1024 : len);
    p->value_split_len = vlen;
    p->value_splits = (max_seqlen + vlen - 1) / vlen;
    p->out_chunks = val_books(h->cfg) * kK / kOutRows;
    p->score_kernel = sliced ? 1 : 0;
    p->score_slice_groups = groups;
    if (fused_values(h->cfg)) p->values = value_shape(h, B, T, max_seqlen, p->value_splits, vlen, stat_len(h, *p));
}

// Carves the workspace.  Array sizes are the larger of what the two score kernels need, so one workspace size serves a batch
// shape whether or not explicit positions are passed.  Behind the statistics, the logits and the partial logits, the score
// stage's arrays and those of the value and output stages share memory: the stages of a call run one after the other, and
// no kernel of one touches what only the other uses.  The latter arrays lie over the partial logits too, except in launches of
// few tokens as far as there is room: lines that other XCDs have just had in their L2 cost the bins' writes 0.8 us (1237
// tokens, 32 + 32 codebooks: 31.7 us a call, 30.9 apart).
void carve(const commvq_handle *h, int B, int64_t T, int max_seqlen, void *base, Workspace *w)
{
    const commvq_config &c = h->cfg;
    Plan pa, pb;
    make_plan(h, B, T, max_seqlen, true, &pa);
    make_plan(h, B, T, max_seqlen, false, &pb);
    if (pair_keys(c)) pb = pa;  // (no explicit positions)
    const size_t ssplits = std::max<size_t>(std::max(pa.score_splits, pb.score_splits), (size_t)stat_splits(h, pa, max_seqlen));
    const size_t vsplits = std::max(pa.value_splits, pb.value_splits);
    const size_t heads = (size_t)B * c.n_q_heads, rows = (size_t)val_books(c) * kK;
    const bool bf16 = c.codebook_dtype == COMMVQ_BF16;
    size_t off = 0;
    auto take = [&](size_t n_floats) {
        float *ptr = base ? reinterpret_cast<float *>(static_cast<char *>(base) + off) : nullptr;
        off += align_up(n_floats * sizeof(float), 256);
        return ptr;
    };
    w->sstat = reinterpret_cast<float2 *>(take(heads * ssplits * 2));
    w->scores = take((size_t)T * c.n_q_heads);
    const size_t parts = bf16 && stream_keys(c) ? (pa.score_slice_groups - 1) * logit_bytes(h, T) : 0;
    const size_t shared = off += parts;
    w->packed = bf16 && !c.position_free ? reinterpret_cast<uint4 *>(take(packed_key_bytes(c) / 4)) : nullptr;
    w->lut = c.position_free ? take(heads * c.m_key * kK) : nullptr;
    const size_t score_end = off, value_bytes = value_stage_bytes(h, B, vsplits);
    off = value_stage_at(shared, parts, score_end - shared, few_tile_bytes(h, B, T, max_seqlen), value_bytes);
    w->vscale = take(heads * vsplits);
    w->lsum = take(heads * vsplits);
    w->bins = reinterpret_cast<unsigned *>(take(heads * vsplits * rows));
    w->partial = take(heads * partial_rows(h, B) * kD);
    w->packed_val = packed_value_room(h, B) ? reinterpret_cast<uint4 *>(take((size_t)c.n_kv_heads * rows * kD * 2 / 4)) : nullptr;
    w->bytes = std::max(off, score_end);
}

// ------------------------------------------------------------------ k_score
struct ScoreDims {
    int Hq, Hkv, nsplit, split_len, n_hi, q_bf16;
    float scale;
};


// Sum over each 16-lane row; every lane of the row receives the row total.
__device__ __forceinline__ float row_sum16(float v)
{
    v += dpp_mov<0xB1>(v);
    v += dpp_mov<0x4E>(v);
    v += dpp_mov<0x141>(v);
    return v + dpp_mov<0x140>(v);
}

// Score kernel.  A wavefront handles FOUR tokens per iteration, one per 16-lane row; lane
// `sub` of a row owns sub-spaces 4*sub .. 4*sub+3 (elements 8*sub .. 8*sub+7), i.e. 16 bytes of
// a bf16 codeword row, so one 16-byte-per-lane buffer load fetches four different codeword
// rows (1 KiB) per instruction: measured ~1.7x the bytes per clock of the one-row-per-
// instruction form, whose rate is bound by the L1's per-instruction cost.  The per-lane byte
// offset (code << 8 | sub * 16) is built by a single byte permute; the codebook index is the
// load's scalar offset.  The relative-position phase is split as 64 * hi + lo: E_hi is folded
// into the query registers (recomputed only when some lane's hi changes, every 64 tokens for
// contiguous positions), E_lo comes from a 32 KiB LDS table.  The dot products are reduced
// inside the 16-lane rows (4 DPP steps per head), parked for 16 iterations and written as
// one 256-byte run per head.  blockIdx.x % Hkv selects the KV head: consecutive workgroups
// go to consecutive XCDs, so with 8 KV heads each XCD's L2 serves one head's codebook.

template <int M, int G, bool BF16>
__global__ __launch_bounds__(kScoreThreads) void k_score(
    const void *__restrict__ q, const uint8_t *__restrict__ key_codes, const void *__restrict__ key_cb,
    const int32_t *__restrict__ cu, const int32_t *__restrict__ q_pos, const int32_t *__restrict__ key_pos,
    const float2 *__restrict__ tbl_hi, const float2 *__restrict__ tbl_lo, float *__restrict__ scores,
    float2 *__restrict__ sstat, const ScoreDims a)
{
    constexpr int CW = M / 4;
    constexpr unsigned ROWB = BF16 ? kD * 2 : kD * 4;
    // E_lo as two planes of float4: plane h, entry [lo][sub] = sub-spaces 4*sub+2h, 4*sub+2h+1
    __shared__ float4 lo_lds[2][kLo][16];
    __shared__ float2 wstat[kScoreThreads / 64][G];

    int id = blockIdx.x;
    const int g = id % a.Hkv;
    id /= a.Hkv;
    const int split = id % a.nsplit;
    const int b = id / a.nsplit;
    const int cu0 = cu[b];
    const int L = cu[b + 1] - cu0;
    const int s0 = split * a.split_len;
    if (s0 >= L) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int r = lane >> 4, sub = lane & 15;
    const int wlen = a.split_len / (kScoreThreads / 64);  // 8, 16, 32 or a multiple of 64 tokens per wavefront (4: launch_score_mg)
    const int t0 = s0 + wave * wlen;
    const int t1 = min(min(t0 + wlen, s0 + a.split_len), L);
    const int n_it = t1 > t0 ? (t1 - t0 + 3) / 4 : 0;
    const int qpos = q_pos[b];

    const uint8_t *codes = key_codes + ((size_t)cu0 * a.Hkv + (size_t)g * L) * M;
    const __amdgpu_buffer_rsrc_t cb_rs =
        make_rsrc(static_cast<const char *>(key_cb) + (size_t)g * M * kK * ROWB, (unsigned)(M * kK) * ROWB);
    const __amdgpu_buffer_rsrc_t hi_rs = make_rsrc(tbl_hi, (unsigned)a.n_hi * kJ * 8u);
    float *srow = scores + (size_t)cu0 * a.Hq + (size_t)g * G * L;
    const size_t q_off = ((size_t)b * a.Hq + (size_t)g * G) * kD + 8 * sub;
    const unsigned sel_lo = opaque_sgpr(0x00003f80u), sel_hi = opaque_sgpr(0x3f800000u);
    const unsigned lane_off = BF16 ? sub * 16u : sub * 32u;

    float qr[G][8];  // queries of the group with E_hi folded in: (x, y) of this lane's 4 sub-spaces
#pragma unroll
    for (int hh = 0; hh < G; ++hh)
#pragma unroll
        for (int e = 0; e < 8; ++e) qr[hh][e] = 0.f;
    int cur_key = -1;  // per lane: (hi << 1 | negative) whose phase is folded into qr
    float keep[G], vmax[G], vsum[G];
#pragma unroll
    for (int hh = 0; hh < G; ++hh) { keep[hh] = 0.f; vmax[hh] = -INFINITY; vsum[hh] = 0.f; }

    // Codeword loads are issued in chunks of CH codebooks into two register buffers; the chunk
    // after the one being summed is always in flight (across iterations too), and the codes
    // are fetched two iterations ahead.
    constexpr int CH = BF16 ? 4 : 2;  // codebooks per chunk
    constexpr int LPC = BF16 ? CH : 2 * CH;                                  // 16-byte loads per chunk
    constexpr int NC = M / CH;
    static_assert(NC % 2 == 0, "buffer parity must repeat every iteration");
    uint4_t buf[2][LPC];
    unsigned cw[CW], cwn[CW];
    auto load_codes = [&](int i, unsigned(&dst)[CW]) {
        const uint4 *cp = reinterpret_cast<const uint4 *>(codes + (size_t)min(i + r, L - 1) * M);
#pragma unroll
        for (int v = 0; v < M / 16; ++v) {
            const uint4 c4 = cp[v];
            dst[4 * v + 0] = c4.x; dst[4 * v + 1] = c4.y; dst[4 * v + 2] = c4.z; dst[4 * v + 3] = c4.w;
        }
    };
    auto issue = [&](const unsigned(&c)[CW], int chunk, uint4_t(&dst)[LPC]) {
#pragma unroll
        for (int k = 0; k < CH; ++k) {
            const int m = chunk * CH + k;
            if (BF16) {
                // byte 1 <- code m, byte 0 <- sub * 16: (code << 8) | (sub * 16)
                const unsigned voff = __builtin_amdgcn_perm(c[m / 4], lane_off, 0x0c0c0000u | ((4u + (m % 4)) << 8));
                dst[k] = __builtin_amdgcn_raw_buffer_load_b128(cb_rs, voff, (unsigned)m * kK * ROWB, 0);
            } else {
                const unsigned voff = ((c[m / 4] >> (8 * (m % 4))) & 0xffu) * ROWB + lane_off;
                dst[2 * k] = __builtin_amdgcn_raw_buffer_load_b128(cb_rs, voff, (unsigned)m * kK * ROWB, 0);
                dst[2 * k + 1] = __builtin_amdgcn_raw_buffer_load_b128(cb_rs, voff + 16u, (unsigned)m * kK * ROWB, 0);
            }
        }
    };
    float A[8];
    auto consume = [&](const uint4_t(&src)[LPC]) {
#pragma unroll
        for (int k = 0; k < LPC; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const unsigned ve = src[k][e];
                if (BF16) {
                    A[2 * e] = add_bf16_sel(ve, sel_lo, A[2 * e]);
                    A[2 * e + 1] = add_bf16_sel(ve, sel_hi, A[2 * e + 1]);
                } else {
                    A[4 * (k & 1) + e] += __builtin_bit_cast(float, ve);
                }
            }
    };
    // the first codes travel while the table is put in place, the first codewords while the others finish theirs
    if (n_it > 0) load_codes(t0, cw);
    for (int x = threadIdx.x; x < 2 * kLo * 16; x += kScoreThreads) {
        const int h = x / (kLo * 16), lo = (x / 16) % kLo, sb = x % 16;
        const float2 e0 = tbl_lo[lo * kJ + 4 * sb + 2 * h], e1 = tbl_lo[lo * kJ + 4 * sb + 2 * h + 1];
        lo_lds[h][lo][sb] = make_float4(e0.x, e0.y, e1.x, e1.y);
    }
    if (n_it > 0) {
        issue(cw, 0, buf[0]);
        load_codes(t0 + 4, cwn);
    }
    __syncthreads();

    for (int it = 0; it < n_it; ++it) {
        const int i = t0 + it * 4;
        // relative position of this row's token
        const int tok = min(i + r, L - 1);
        const int pos = key_pos ? key_pos[cu0 + tok] : tok;
        const int dl = qpos - pos;
        const int neg = dl < 0;
        const int ad = neg ? -dl : dl;
        const int hi = min(ad >> kLoBits, a.n_hi - 1);
        const int lo = ad & (kLo - 1);
        const int key = (hi << 1) | neg;
        if (__builtin_amdgcn_ballot_w64(key != cur_key) != 0) {
            // fold the coarse phase into the queries: q' = q conj(E_hi) for t >= p, q E_hi otherwise
            cur_key = key;
            float eh[8];
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
                const uint4_t v = __builtin_amdgcn_raw_buffer_load_b128(hi_rs, (unsigned)hi * (kJ * 8u) + sub * 32u + 16u * hf, 0, 0);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const unsigned ve = v[e];
                    eh[4 * hf + e] = __builtin_bit_cast(float, ve);
                }
            }
#pragma unroll
            for (int hh = 0; hh < G; ++hh) {
                float qx[4], qy[4];
                if (a.q_bf16) {
                    const uint4 v = *reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(q) + q_off + (size_t)hh * kD);
                    const unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) { qx[e] = bf16_lo(w[e]) * a.scale; qy[e] = bf16_hi(w[e]) * a.scale; }
                } else {
                    const float4 *qp = reinterpret_cast<const float4 *>(static_cast<const float *>(q) + q_off + (size_t)hh * kD);
                    const float4 v0 = qp[0], v1 = qp[1];
                    qx[0] = v0.x * a.scale; qy[0] = v0.y * a.scale; qx[1] = v0.z * a.scale; qy[1] = v0.w * a.scale;
                    qx[2] = v1.x * a.scale; qy[2] = v1.y * a.scale; qx[3] = v1.z * a.scale; qy[3] = v1.w * a.scale;
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float hc = eh[2 * e], hs = neg ? -eh[2 * e + 1] : eh[2 * e + 1];
                    qr[hh][2 * e] = qx[e] * hc + qy[e] * hs;
                    qr[hh][2 * e + 1] = qy[e] * hc - qx[e] * hs;
                }
            }
        }
        // A = sum of the M selected codeword rows (Eq. commute_decode), this lane's 4 sub-spaces
#pragma unroll
        for (int e = 0; e < 8; ++e) A[e] = 0.f;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            // (the last iteration issues one redundant, in-range chunk rather than branch)
            if (c + 1 < NC) issue(cw, c + 1, buf[(c + 1) & 1]);
            else issue(cwn, 0, buf[0]);
            __builtin_amdgcn_sched_barrier(0);
            consume(buf[c & 1]);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int v = 0; v < CW; ++v) cw[v] = cwn[v];
        load_codes(i + 8, cwn);  // token index is clamped to the sequence

        // B = A E_lo (conjugated for negative distances); score_h = sum_j Re(q'_h conj(B))
        const float4 l0 = lo_lds[0][lo][sub], l1 = lo_lds[1][lo][sub];
        const float ec[4] = {l0.x, l0.z, l1.x, l1.z};
        const float es[4] = {neg ? -l0.y : l0.y, neg ? -l0.w : l0.w, neg ? -l1.y : l1.y, neg ? -l1.w : l1.w};
        float Bx[4], By[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            Bx[e] = A[2 * e] * ec[e] - A[2 * e + 1] * es[e];
            By[e] = A[2 * e] * es[e] + A[2 * e + 1] * ec[e];
        }
        const bool mine = sub == (it & 15);
#pragma unroll
        for (int hh = 0; hh < G; ++hh) {
            float v = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) v += qr[hh][2 * e] * Bx[e] + qr[hh][2 * e + 1] * By[e];
            v = row_sum16(v);
            keep[hh] = mine ? v : keep[hh];
        }
        if ((it & 15) == 15 || it == n_it - 1) {  // flush: lane (r, sub) holds token 4 * sub + r of this 64-token block
            const int itc = (it & ~15) + sub;
            const int tk = t0 + itc * 4 + r;
            if (itc <= it && tk < t1) {
#pragma unroll
                for (int hh = 0; hh < G; ++hh) {
                    srow[(size_t)hh * L + tk] = keep[hh];
                    const float mn = fmaxf(vmax[hh], keep[hh]);
                    vsum[hh] = vsum[hh] * __builtin_amdgcn_exp2f((vmax[hh] - mn) * kLog2e) +
                               __builtin_amdgcn_exp2f((keep[hh] - mn) * kLog2e);
                    vmax[hh] = mn;
                }
            }
        }
    }

    // (max, sum exp) of the split: lanes -> waves -> one pair per head
#pragma unroll
    for (int hh = 0; hh < G; ++hh) {
        const float m = wave_max(vmax[hh]);
        const float l = wave_sum(vmax[hh] == -INFINITY ? 0.f : vsum[hh] * __builtin_amdgcn_exp2f((vmax[hh] - m) * kLog2e));
        if (lane == 0) wstat[wave][hh] = make_float2(m, l);
    }
    __syncthreads();
    if (threadIdx.x < G) {
        float m = -INFINITY;
        for (int w = 0; w < kScoreThreads / 64; ++w) m = fmaxf(m, wstat[w][threadIdx.x].x);
        float l = 0.f;
        for (int w = 0; w < kScoreThreads / 64; ++w) {
            const float2 st = wstat[w][threadIdx.x];
            if (st.x != -INFINITY) l += st.y * __builtin_amdgcn_exp2f((st.x - m) * kLog2e);
        }
        sstat[((size_t)b * a.Hq + (size_t)g * G + threadIdx.x) * a.nsplit + split] = make_float2(m, l);
    }
}

// ------------------------------------------------------------------ k_score_few
// k_score for launches that leave a wavefront no more than four tokens, one per 16-lane row: nothing is gone round, so nothing is
// pipelined from one iteration to the next and the E_lo table does not pay for its way into LDS (32 KB a workgroup, against 8 KB of
// rows a token).  Everything that does not depend on the codes (queries, phase factors) is asked for first, then the rows of all
// codebooks, at most 48 16-byte pieces a lane at once: with 8 at a time, as in k_score, a wavefront alone on its SIMD waits for
// every group of them.  The grid has a dimension for each of head, tile and sequence, which saves the divisions.
// Bound by latency (arguments, sequence, codes, rows, one after the other) and by the rows' way through the L1s, 48 bytes a clock and compute
// unit.  Whole calls with k_score and with this, in microseconds: one fp32 head of 4096 tokens, 32 + 32 codebooks 18.8 -> 15.9 (64 MB of
// rows, 3 us of them); 8 x 4 heads, explicit positions, 16 + 16 codebooks 1237 tokens 17.1 -> 14.9, 4000 26.3 -> 20.6; 32 + 32 codebooks 1237
// tokens 22.3 -> 19.6, 4000 33.3 -> 28.8.
template <int M, int G, bool BF16>
__global__ __launch_bounds__(kScoreThreads) void k_score_few(
    const void *__restrict__ q, const uint8_t *__restrict__ key_codes, const void *__restrict__ key_cb,
    const int32_t *__restrict__ cu, const int32_t *__restrict__ q_pos, const int32_t *__restrict__ key_pos,
    const float2 *__restrict__ tbl_hi, const float2 *__restrict__ tbl_lo, float *__restrict__ scores,
    float2 *__restrict__ sstat, const ScoreDims a)
{
    constexpr unsigned ROWB = BF16 ? kD * 2 : kD * 4;
    constexpr int QL = 2;                                     // 16-byte pieces of a query head at most
    constexpr int PC = BF16 ? 1 : 2;                          // 16-byte pieces of a codeword that a lane takes
    constexpr int DEPTH = M * PC <= 48 ? M : 48 / PC;         // codebooks whose rows are in flight
    typedef unsigned u4u __attribute__((ext_vector_type(4), aligned(2)));  // (queries and codebooks: any alignment that their elements have)
    __shared__ float logit[G][kFewTokens];

    const int g = blockIdx.x, split = blockIdx.y, b = blockIdx.z;
    const int cu0 = cu[b], L = cu[b + 1] - cu0, qpos = q_pos[b];
    asm volatile("" ::"s"(qpos));                             // (asked for here, with the others)
    const int s0 = split * kFewTokens;
    if (s0 >= L) return;
    const int tid = threadIdx.x, lane = tid & 63, sub = lane & 15;
    const int tok = min(s0 + (tid >> 4), L - 1);
    int pos = tok;                                            // (asked for first: a wait for it is not one for the codes)
    if (key_pos) pos = key_pos[cu0 + tok];
    __builtin_amdgcn_sched_barrier(0);

    unsigned cw[M / 4];
    {
        const uint4 *cp = reinterpret_cast<const uint4 *>(key_codes + ((size_t)cu0 * a.Hkv + (size_t)g * L + tok) * M);
#pragma unroll
        for (int v = 0; v < M / 16; ++v) {
            const uint4 c4 = cp[v];
            cw[4 * v + 0] = c4.x; cw[4 * v + 1] = c4.y; cw[4 * v + 2] = c4.z; cw[4 * v + 3] = c4.w;
        }
    }
    const int dl = qpos - pos;
    const bool neg = dl < 0;
    const int ad = neg ? -dl : dl;
    const int hi = min(ad >> kLoBits, a.n_hi - 1), lo = ad & (kLo - 1);
    const __amdgpu_buffer_rsrc_t hi_rs = make_rsrc(tbl_hi, (unsigned)a.n_hi * kJ * 8u), lo_rs = make_rsrc(tbl_lo, (unsigned)kLo * kJ * 8u);
    uint4_t ph[2][2];                                         // coarse and fine phase factors of the lane's 4 sub-spaces
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
        ph[0][hf] = __builtin_amdgcn_raw_buffer_load_b128(hi_rs, (unsigned)hi * (kJ * 8u) + sub * 32u + 16u * hf, 0, 0);
        ph[1][hf] = __builtin_amdgcn_raw_buffer_load_b128(lo_rs, (unsigned)lo * (kJ * 8u) + sub * 32u + 16u * hf, 0, 0);
    }
    uint4_t qw[G][QL];
    {
        const unsigned qb = a.q_bf16 ? 2u : 4u, next = a.q_bf16 ? 0u : 16u;  // (bf16: the same piece twice, no branch)
        const char *qp = static_cast<const char *>(q) + ((size_t)b * a.Hq + (size_t)g * G) * kD * qb;
#pragma unroll
        for (int hh = 0; hh < G; ++hh) {
            qw[hh][0] = *reinterpret_cast<const u4u *>(qp + (hh * kD + 8 * sub) * qb);
            qw[hh][1] = *reinterpret_cast<const u4u *>(qp + (hh * kD + 8 * sub) * qb + next);
        }
    }
    __builtin_amdgcn_sched_barrier(0);

    const char *cb0 = static_cast<const char *>(key_cb) + (size_t)g * M * kK * ROWB;
    const unsigned lane_off = BF16 ? sub * 16u : sub * 32u;
    uint4_t row[M][PC];
    auto issue = [&](int m) __attribute__((always_inline)) {
        if (BF16) {
            // byte 1 <- code m, byte 0 <- sub * 16: (code << 8) | (sub * 16)
            const unsigned voff = __builtin_amdgcn_perm(cw[m / 4], lane_off, 0x0c0c0000u | ((4u + (m % 4)) << 8));
            row[m][0] = *reinterpret_cast<const u4u *>(cb0 + (size_t)m * kK * ROWB + voff);
        } else {
            const unsigned voff = ((cw[m / 4] >> (8 * (m % 4))) & 0xffu) * ROWB + lane_off;
#pragma unroll
            for (int p = 0; p < PC; ++p) row[m][p] = *reinterpret_cast<const u4u *>(cb0 + (size_t)m * kK * ROWB + 16 * p + voff);
        }
    };
    const unsigned sel_lo = opaque_sgpr(0x00003f80u), sel_hi = opaque_sgpr(0x3f800000u);
    float A[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) A[e] = 0.f;
#pragma unroll
    for (int m = 0; m < DEPTH; ++m) issue(m);
    __builtin_amdgcn_sched_barrier(0);
    // the phase of the relative position (conjugated for keys behind the query)
    float ex[4], ey[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const unsigned hxr = ph[0][u / 2][2 * (u % 2)], hyr = ph[0][u / 2][2 * (u % 2) + 1];
        const unsigned lxr = ph[1][u / 2][2 * (u % 2)], lyr = ph[1][u / 2][2 * (u % 2) + 1];
        const float hx = __builtin_bit_cast(float, hxr), hy = __builtin_bit_cast(float, hyr);
        const float lx = __builtin_bit_cast(float, lxr), ly = __builtin_bit_cast(float, lyr);
        ex[u] = hx * lx - hy * ly;
        const float y = hx * ly + hy * lx;
        ey[u] = neg ? -y : y;
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m0 = 0; m0 < M; m0 += 4) {
#pragma unroll
        for (int m = m0; m < m0 + 4; ++m)
#pragma unroll
            for (int p = 0; p < PC; ++p)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const unsigned ve = row[m][p][e];
                    if (BF16) {
                        A[2 * e] = add_bf16_sel(ve, sel_lo, A[2 * e]);
                        A[2 * e + 1] = add_bf16_sel(ve, sel_hi, A[2 * e + 1]);
                    } else {
                        A[4 * p + e] += __builtin_bit_cast(float, ve);
                    }
                }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = m0 + DEPTH; m < m0 + DEPTH + 4; ++m)
            if (m < M) issue(m);
        __builtin_amdgcn_sched_barrier(0);
    }
    // B = A E, score_h = sum_j Re(q_h conj(B))
    float B[8];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        B[2 * u] = A[2 * u] * ex[u] - A[2 * u + 1] * ey[u];
        B[2 * u + 1] = A[2 * u] * ey[u] + A[2 * u + 1] * ex[u];
    }
#pragma unroll
    for (int hh = 0; hh < G; ++hh) {
        float v = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const unsigned wb = qw[hh][0][e / 2], wf = qw[hh][e / 4][e % 4];
            const float x = a.q_bf16 ? (e & 1 ? bf16_hi(wb) : bf16_lo(wb)) : __builtin_bit_cast(float, wf);
            v += x * a.scale * B[e];
        }
        v = row_sum16(v);
        if (sub == 0) logit[hh][tid >> 4] = v;
    }
    __syncthreads();
    // logits, and (max, sum of exp) of the workgroup's tokens: 16 lanes per head
    if (tid < G * kFewTokens) {
        const int hh = tid / kFewTokens, t = s0 + tid % kFewTokens;
        const float v = t < L ? logit[hh][tid % kFewTokens] : -INFINITY;
        if (t < L) scores[(size_t)cu0 * a.Hq + (size_t)(g * G + hh) * L + t] = v;
        float m = v;
        m = fmaxf(m, dpp_mov<0xB1>(m));
        m = fmaxf(m, dpp_mov<0x4E>(m));
        m = fmaxf(m, dpp_mov<0x141>(m));
        m = fmaxf(m, dpp_mov<0x140>(m));
        const float l = row_sum16(v == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((v - m) * kLog2e));
        if (tid % kFewTokens == 0) sstat[((size_t)b * a.Hq + (size_t)g * G + hh) * a.nsplit + split] = make_float2(m, l);
    }
}

// ------------------------------------------------------------------ k_prep
constexpr int kSliceThreads = 1024;              // one workgroup per compute unit

// Key codebook re-laid for k_score_stream.
//   packed[g][s][blk][c][col] : 16-byte pieces (8 bf16).  Slice s holds elements 8 s .. 8 s + 7 of every codeword as
//                        one (M = 16) or two (M = 32) contiguous 64 KiB images of 256 rows (one per code value c) x 16
//                        pieces: codebook 16 blk + col.  A 256-byte row spans all 64 LDS banks, so a piece
//                        lives in bank column col whatever its code: lanes that read different columns never conflict.
// One thread per 16-byte piece of the source (coalesced reads).
__global__ __launch_bounds__(256) void k_prep(const uint4 *__restrict__ key_cb, uint4 *__restrict__ packed, int Hkv, int M)
{
    const size_t n_pieces = (size_t)Hkv * M * kK * 16;
    const size_t t = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= n_pieces) return;
    const int sl = (int)(t & 15);               // a row's 16 pieces of 8 elements: one per slice
    const size_t row = t >> 4;                  // (g * M + m) * K + c
    const int g = (int)(row / ((size_t)M * kK));
    const int mc = (int)(row % ((size_t)M * kK));
    const int m = mc / kK, c = mc % kK;
    packed[(((size_t)g * 16 + sl) * (M / 16) + m / 16) * (kK * 16) + c * 16 + m % 16] = key_cb[t];
}

struct SliceDims {
    int Hq, Hkv, nsplit, n_hi, q_bf16;
    float scale;
};

// ------------------------------------------------------------------ k_score_stream

// 16-byte LDS read at an absolute LDS byte address.  The score kernels keep their dynamic LDS at address 0
// (no static LDS), but the compiler only learns that after instruction selection: a read through the array's
// base costs one "add 0" per read.
typedef __attribute__((address_space(3))) const uint4_t *lds_u4_ptr;
typedef __attribute__((address_space(3))) const uint2_t *lds_u2_ptr;
__device__ __forceinline__ uint4_t lds_read_b128(unsigned byte_addr) { return *reinterpret_cast<lds_u4_ptr>(byte_addr); }

// Workgroup barrier that waits for nothing by itself: the caller has waited for what the others may rely on (LDS
// reads that have been consumed, lds_dma16 loads by s_waitcnt).  No LDS access moves across it.
__device__ __forceinline__ void bare_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

constexpr int kBlockBytes = 64 * 1024;    // 16 codebooks x 256 codewords x 16 bytes
// LDS behind the two 64 KiB blocks, per buffer of two, in 16-byte pieces (what a slice needs besides the codebook, sent
// from memory straight into LDS by thread x to piece x): fine phase factors [2 parts][64], coarse ones [8 passes][9 rows]
// [2 parts] padded to whole wavefronts, raw queries [8 passes][G heads][1 (bf16) or 2 (fp32)]
constexpr int kAuxHi = 2 * kLo, kAuxQ = kAuxHi + 192, kAuxPieces = kAuxQ + 128;
constexpr int kHiRows = 9;
constexpr int kAuxBytes = kAuxPieces * 16;
constexpr int kSegOff = 2 * kBlockBytes + 2 * kAuxBytes;          // int4 per pass: sequence, first token, length, cu_seqlens
constexpr int kWstOff = kSegOff + kStreamPasses * 16;             // float2 [8 passes][2 halves][8 heads]
constexpr int kAuxTabOff = kWstOff + kStreamPasses * 2 * 8 * 8;   // where thread x's piece comes from (for slice 0)
constexpr int kStreamLds = kAuxTabOff + kAuxPieces * 8;
constexpr int kPairLds = 129696;                                  // k_score_pair's

struct StreamDims {
    int Hq, Hkv, G, batch, n_hi, q_bf16;
    float scale;
    int tiles;             // workgroups per KV head and slice group
    int groups;            // workgroups per tile, each with S / groups of the codebook slices
    int nstat;             // 512-token statistics per (sequence, query head)
    long long part_stride; // floats between the partial logit arrays of two slice groups
};

// Slice-streaming score kernel with both contractions on the matrix cores (Eq. new_attention,
// re-bracketed: gather-sum the codeword blocks first, rotate once, contract with the G queries).
// Works on the key codebook repacked by k_prep: slice sl = 8 consecutive elements of every codeword, as one (M = 16) or
// two (M = 32) 64 KiB LDS images of 256 rows (code value) x 16 bank columns (codebook).
//
// Tokens.  The contexts of a KV head, one sequence after the other, are cut into segments of 512 tokens; a workgroup takes
// `passes` consecutive segments -- of one long sequence, or of several short ones: everything that depends on the sequence
// (query, distances, output place) is looked up per pass.  A pass is 64 fine positions (token mod 64) x 8 coarse rows; a
// wavefront owns 4 fine positions, and lane n of its 16 token lanes takes fine position n / 4 and coarse rows n % 4 (set 0)
// and 4 + n % 4 (set 1).  So the four lanes of a 4-lane block, both sets and all passes of one sequence are whole coarse
// rows (64 tokens) apart: they share the fine phase factor E_lo of the relative position 64 H + lo, which is folded
// into the block's query operand once per slice, and a pass only rotates by the coarse factor E_hi.
//
// Codes.  The tile's codes are read once and stay in registers for all slices, in the byte order of the lane's gather steps.
//
// Per slice and pass:
//  1. Gather-sum: v_smfmac_f32_16x16x64_bf16 (structured-sparse first operand) with a constant 0/1 selection
//     matrix as first operand and 128 gathered pieces as second: lane n + 16 g supplies two pieces, A for token n
//     of set 0 and B for token n of set 1, of the same codebook.  Products with 1.0 are exact, so this is the plain fp32 sum
//     of the M codeword slices.  Rows 0..7 of the result are elements 0..7 of set 0's tokens, rows 8..15 those of set 1's:
//     lane (n, g) receives elements 4 (g & 1) .. + 3 of its token of set g >> 1.
//     The LDS reads of a group of steps are issued right after the matrix instructions that consumed the
//     group's registers, so the first reads of the next pass travel while this pass is finished.
//  2. Each lane rotates its two (x, y) sub-spaces by the coarse phase factor of its token.
//  3. Contraction with the queries.  The two lanes of a token hold half of its 8 elements each.  Logits are sums over
//     elements, so each lane keeps the sum of its own half for all slices, and the two meet once, at the write-out: four chained
//     v_mfma_f32_4x4x1_16b_f32 (in a block of 4 lanes, lane i supplies q'[head i][element], every lane its own element) add a
//     pass's whole contribution to the accumulators of 4 heads, and the query operand is folded for 4 elements instead of 8.  They run between
//     the steps of the next pass.  With two groups of heads (8) there are no registers for accumulators of every pass: there
//     an exchange of 16-lane rows between the passes of a pair (4 v_permlane16_swap) gives the even lane all 8 elements of its
//     token of the even pass and the odd lane those of the odd pass, and eight chained instructions per group follow.  For 4 heads
//     that, and the next slice of M = 32 through registers that the halves need: 128K tokens, M = 16 82.5 against 80.2 us a call, 8 x
//     8K..64K, M = 32 457 against 434, 32K 55.7 against 54.4, 64 x 512..1024 115 against 110; rms error of the logits against 64 bits
//     1.25e-7 and 1.06e-7 (M = 16), 1.58e-7 and 1.25e-7 (M = 32).
// What bounds it: LDS and SIMD issue.  With four wavefronts on a SIMD a sparse MFMA takes 17 clk of it, a 4x4x1 one 9, a row swap 9,
// a byte permute 5, a rotation's multiplication or addition 3 to 4 (micro-benchmark), and they add up; a pass is 4 (8) + 5 + 8 (16)
// + 8 of these for M = 16 (32) and 4 heads = 180 (290) clk, and the compute unit's LDS needs 4.35 clk for each of the M / 2 + 1
// 16-byte reads of its 16 wavefronts and 8 for each KiB of the next slice, 173 (332) per SIMD and pass.  Measured per pass: 223 (398) clk, at
// 2.2 GHz; the rest is the switch of slices and what the latencies of one wavefront's chain leave open.  (With 8 heads 440 for M = 32.)
// A wavefront that is behind issues first (s_setprio by pass), pass by pass in the last ones: waves that run ahead leave the last ones
// alone on their SIMD before each barrier (one level per two passes instead: 8 x 8K..64K 458.5 us, 454.2 so; 128K 82.8 and 82.0).
//
// Slices.  M = 16: the two 64 KiB blocks take slices in turn, the next one travels (memory -> LDS, no registers)
// while the current one is worked on: one barrier per slice.  Its sends are spread over the passes, since a burst fills
// the memory pipe's queue and stops the wavefronts for up to 2000 clk.  M = 32: a slice fills both blocks (codebooks 0..15 |
// 16..31).  Its last pass is done with block 0 after half of its steps and with block 1 at its end; the next slice's are sent for
// right then, and block 1 is waited for after the first half of the next slice's first pass.  (Block 1 sent for behind the barrier between the
// slices, which saves one: 8 x 8K..64K 437 -> 443.)  8 heads with M = 32 and eight passes spill 6 registers.
//
// Not kept: three or four steps of reads in flight instead of two (no change, or spills); M = 32 as two sweeps of 16 codebooks with the
// gather sums carried in registers, which allows double buffering but only 4 to 6 passes (8 heads: 549 us instead of 475).
//
// Short contexts: a launch may cut every tile along the slices as well (StreamDims::groups workgroups per
// tile); each then writes partial logits, which k_score_combine adds.
//
// FORM: 1 up to 4 heads, logits in halves; 0 up to 4 heads, rows exchanged in pairs of passes (exchange_rows); 2 eight heads, likewise.
template <int M, int FORM, int NP>
__global__ __launch_bounds__(kSliceThreads) void k_score_stream(
    const void *__restrict__ q, const uint8_t *__restrict__ key_codes, const uint4 *__restrict__ packed,
    const int32_t *__restrict__ cu, const int32_t *__restrict__ q_pos, const float2 *__restrict__ tbl_hi,
    const float2 *__restrict__ tbl_lo, float *__restrict__ scores, float2 *__restrict__ sstat, const StreamDims a)
{
    constexpr int S = kStreamSlices;
    constexpr int NB = M / 16;                                // 64 KiB blocks per slice
    constexpr int NST = 4 * NB;                               // gather steps (sparse matrix instructions) per pass
    constexpr int NGRP = FORM == 2 ? 2 : 1;
    const int G = NGRP == 2 ? 8 : a.G;                        // query heads of the KV head; NGRP groups of 4, padded with zero queries
    constexpr int NBUF = 2;                                   // gather steps whose LDS reads are in flight
    constexpr bool HALF = FORM == 1;                          // logits in two halves, each of the elements that a lane has (8 heads: no registers)
    extern __shared__ __attribute__((aligned(16))) uint4 tab[];

    int id = blockIdx.x;
    const int g = id % a.Hkv;                                 // (head = index mod Hkv: with 8 KV heads an XCD serves one head)
    id /= a.Hkv;
    const int tile = id % a.tiles;
    const int eg = id / a.tiles;                              // which group of slices
    const int s_begin = eg * (S / a.groups), s_end = s_begin + S / a.groups;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // The slice's codebook images: thread x's piece x of every 16 KiB, memory -> LDS.
    const char *src = reinterpret_cast<const char *>(packed) + (size_t)g * S * NB * kBlockBytes;
    auto send_part = [&](int sl, int blk, int slot, int j) {
        const char *p = src + ((size_t)sl * NB + blk) * kBlockBytes + j * 16384;
        lds_dma16(p, (unsigned)(wave * 64 + fresh_lane()) * 16u, (unsigned)(slot * kBlockBytes + j * 16384 + wave * 1024));
    };
    auto send_block = [&](int sl, int blk, int slot) {
#pragma unroll
        for (int j = 0; j < 4; ++j) send_part(sl, blk, slot, j);
    };
    send_block(s_begin, 0, M == 16 ? s_begin & 1 : 0);
    if (M == 32) send_block(s_begin, 1, 1);

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
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // the blocks sent for above have landed
        return;
    }
    unsigned chg = 1u;                                        // bit p: pass p is of another sequence than pass p - 1
    bool neg = false;                                         // some distance is negative
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        if (p > 0 && p < np && pb[p] != pb[p - 1]) chg |= 1u << p;
        if (p < np && qd[p] < kPassTokens - 1) neg = true;
    }

    const int n = lane & 15, gk = lane >> 4;
    const int par = gk & 1, hi = gk >> 1;                     // par: half of the 8 elements; hi: set of 16 tokens
    const int f = 4 * wave + (n >> 2);                        // fine position

    // The tile's codes: every lane asks for what no other asks for, 8 bytes (M = 16: bytes 8 par .. + 7) or 16 (M = 32: block
    // par) of its token of set hi; the lanes exchange the rest below.
    constexpr int RAW = M / 8;
    unsigned raw[NP][RAW];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        // tokens past the end of the sequence read zeros (the descriptor ends with the sequence): code 0, a valid row
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(key_codes + ((size_t)pcu[p] * a.Hkv + (size_t)g * pL[p]) * M, p < np ? (unsigned)pL[p] * M : 0u);
        const unsigned at = (unsigned)(pt0[p] + f + kLo * ((n & 3) + 4 * hi)) * M + (M == 16 ? 8u : 16u) * par;
        if (M == 16) {
            const uint2_t c = __builtin_amdgcn_raw_buffer_load_b64(rs, at, 0, 0);
            raw[p][0] = c[0]; raw[p][1] = c[1];
        } else {
            const uint4_t c = __builtin_amdgcn_raw_buffer_load_b128(rs, at, 0, 0);
#pragma unroll
            for (int i = 0; i < RAW; ++i) raw[p][i] = c[i & 3];
        }
    }

    // What a slice needs besides the codebook: thread x < kAuxPieces sends for piece x.  The source of its piece of slice 0
    // waits in LDS between the slices (bit 0 of a coarse factor's: take the conjugate, the row's distance is negative).
    unsigned long long *aux_tab = reinterpret_cast<unsigned long long *>(reinterpret_cast<char *>(tab) + kAuxTabOff);
    {
        uintptr_t aux = 0;
        if (tid < kAuxHi) {
            aux = reinterpret_cast<uintptr_t>(tbl_lo + (size_t)(tid % kLo) * kJ + 2 * (tid / kLo));
        } else if (tid < kAuxQ) {
            const int x = tid - kAuxHi, p = x / (2 * kHiRows), row = x % (2 * kHiRows) / 2;
            int D = 0;
#pragma unroll
            for (int k = 0; k < NP; ++k)
                if (p == k) D = qd[k];
            const int H = ((D + 1) >> kLoBits) - 8 + row;     // rows 0..8: what distances D - 511 .. D can reach
            if (p < np) aux = reinterpret_cast<uintptr_t>(tbl_hi + (size_t)min(H < 0 ? -H : H, a.n_hi - 1) * kJ + 2 * (x & 1)) | (H < 0 ? 1u : 0u);
        } else if (tid < kAuxPieces) {
            const int x = tid - kAuxQ, per = a.q_bf16 ? 1 : 2;
            const int p = x / (G * per), h = x / per % G, part = x % per;
            int bs = 0;
#pragma unroll
            for (int k = 0; k < NP; ++k)
                if (p == k) bs = pb[k];
            if (p < np) aux = reinterpret_cast<uintptr_t>(q) + (((size_t)bs * a.Hq + (size_t)g * G + h) * kD * (a.q_bf16 ? 2 : 4) + part * 16);
        }
        if (tid < kAuxPieces) aux_tab[tid] = aux;
    }
    const bool q_odd = (reinterpret_cast<uintptr_t>(q) & 15u) != 0;
    auto send_aux = [&](int sl, int buf) {
        if (wave >= kAuxPieces / 64) return;
        const int x = wave * 64 + fresh_lane();
        const uintptr_t aux = aux_tab[x];
        if (!aux) return;
        const unsigned step = wave >= kAuxQ / 64 && a.q_bf16 ? 16u : 32u;
        char *dst = reinterpret_cast<char *>(tab) + 2 * kBlockBytes + buf * kAuxBytes + x * 16;
        if (neg && wave >= kAuxHi / 64 && wave < kAuxQ / 64) {  // the conjugate of the row of |H| needs a register
            float4 e = *reinterpret_cast<const float4 *>((aux & ~(uintptr_t)1) + sl * step);
            if (aux & 1) { e.y = -e.y; e.w = -e.w; }
            *reinterpret_cast<float4 *>(dst) = e;
        } else if (q_odd && wave >= kAuxQ / 64) {              // queries that are not 16-byte aligned
            const uint16_t *e = reinterpret_cast<const uint16_t *>(aux + sl * step);
            for (int k = 0; k < 8; ++k) reinterpret_cast<uint16_t *>(dst)[k] = e[k];
        } else {
            lds_dma16(reinterpret_cast<const void *>(aux + sl * step), (unsigned)(2 * kBlockBytes + buf * kAuxBytes + wave * 1024));
        }
    };
    send_aux(s_begin, s_begin & 1);

    // Selection operand of v_smfmac_f32_16x16x64_bf16 (first operand structured-sparse: two of every four
    // consecutive k kept, 2-bit positions in an index register).  Its second operand takes two 16-byte pieces per
    // lane, A (elements 0..7) and B (8..15); measured layout (micro-benchmark smfmac_layouts): logical k =
    // 32 * (A | B) + 8 * (lane / 16) + element, and first-operand lane (row i, block q) covers k = 16 q .. 16 q + 15
    // with stored slots 2 t, 2 t + 1 for its t-th group of four.  Rows 0..7 must add element i of the four lanes'
    // A pieces, rows 8..15 element i - 8 of their B pieces: lane (i, q) is active when (i < 8) == (q < 2) and then
    // keeps 1.0 at position e % 4 of groups e / 4 and 2 + e / 4 (e = i % 8); every other stored value is 0.0.
    uint4_t sel = {0u, 0u, 0u, 0u};
    unsigned sidx = 0x44444444u;  // default positions (0, 1) of every stored pair
    {
        const int e = n & 7;
        if ((n < 8) == (gk < 2)) {
            const int t = e >> 2, pos = e & 3, other = pos == 0 ? 1 : 0;
            sel[t] = 0x00003f80u;        // slot 2 t      = 1.0, slot 2 t + 1 = 0.0
            sel[2 + t] = 0x00003f80u;    // slot 4 + 2 t  = 1.0
            const unsigned pair = (unsigned)pos | (unsigned)other << 2;
            sidx = (sidx & ~(0xfu << (4 * t)) & ~(0xfu << (4 * (2 + t)))) | pair << (4 * t) | pair << (4 * (2 + t));
            sidx = (sidx & 0xffffu) | sidx << 16;
        }
    }
    const bf16x8_t selv = __builtin_bit_cast(bf16x8_t, sel);

    // What a lane gathers, for tokens n of both sets: the 4 codebooks 8 par + (n + 4 hi + st) mod 8, st = 0..3, of every
    // block of 16; the four lanes of a token cover the block.  In every group of lanes that the LDS checks
    // against each other for bank conflicts the 16 pieces of one read then come from 16 different bank columns,
    // whatever the codes.  xreg[st]: byte 0 = 16 * column read at step st, bytes 2 and 3 = 0 and 1; a byte permute splices the
    // code in as byte 1 and byte 2 or 3 as byte 2, which yields the LDS byte address 65536 slot + 256 c + 16 col.
    unsigned xreg[4];
#pragma unroll
    for (int st = 0; st < 4; ++st) xreg[st] = (unsigned)(8 * par + ((n + st + 4 * hi) & 7)) * 16u | 1u << 24;
    unsigned rsel = 0u;  // byte selector that rotates 8 code bytes so that step st finds its code at byte st
#pragma unroll
    for (int x = 0; x < 4; ++x) rsel |= (unsigned)((x + n + 4 * hi) & 7) << (8 * x);

    // ccall[p][v][blk]: the code bytes of steps 4 blk .. + 3 for the lane's token of set v, pass p
    unsigned ccall[NP][2][NB];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        unsigned d[2][2 * NB];                                // both sets' tokens: bytes 8 par .. + 7 of every block of 16
        unsigned own[2 * NB];
        if (M == 16) {
            own[0] = raw[p][0]; own[1] = raw[p][1];
        } else {                                              // rows exchanged: halves of both blocks instead of one block
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                auto r = __builtin_amdgcn_permlane16_swap(raw[p][i], raw[p][(2 + i) % RAW], false, false);
                own[i] = r[0];
                own[(2 + i) % (2 * NB)] = r[1];
            }
        }
#pragma unroll
        for (int i = 0; i < 2 * NB; ++i) {                    // lower half of the wavefront: set 0, upper half: set 1
            auto r = __builtin_amdgcn_permlane32_swap(own[i], own[i], false, false);
            d[0][i] = r[0];
            d[1][i] = r[1];
        }
#pragma unroll
        for (int v = 0; v < 2; ++v)
#pragma unroll
            for (int k = 0; k < NB; ++k) ccall[p][v][k] = __builtin_amdgcn_perm(d[v][2 * k + 1], d[v][2 * k], rsel);
    }
    if (wave == 0 && lane < NP) {                             // the segments, for the write-out
        int4 s = make_int4(0, 0, 0, 0);
#pragma unroll
        for (int p = 0; p < NP; ++p)
            if (lane == p) s = make_int4(pb[p], pt0[p], pL[p], pcu[p]);
        reinterpret_cast<int4 *>(reinterpret_cast<char *>(tab) + kSegOff)[lane] = s;
    }

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
    float qrow[NGRP][HALF ? 4 : 8];                                      // q' of the slice: head 4 x + n % 4, the 8 elements
    unsigned ehi_at = 0u;                                     // LDS address of the lane's coarse factor in pass 0's rows
    // where the lane finds its fine and coarse factor of pass 0's sequence, from the start of a buffer: bits 0..15, 16..31
    unsigned at0;
    {
        const int D0 = qd[0], D1 = qd[NP > 1 ? 1 : 0], ln = fresh_lane(), fl = 4 * wave + (ln >> 2 & 3), Dl = ln >> 4 & 1 ? D1 : D0;
        const int row = ((D0 - fl) >> kLoBits) - ((D0 + 1) >> kLoBits) + 8 - (ln & 3) - 4 * (ln >> 5);
        at0 = (unsigned)(HALF ? ((D0 - fl) & (kLo - 1)) + (ln >> 4 & 1) * kLo : (Dl - fl) & (kLo - 1)) * 16u | (unsigned)(kAuxHi + 2 * row + (ln >> 4 & 1)) << 20;
    }
    for (int sl = s_begin; sl < s_end; ++sl) {
        const bool more = sl + 1 < s_end;
        const int buf = sl & 1;
        const unsigned aux0 = (unsigned)(2 * kBlockBytes + buf * kAuxBytes);
        // this slice (M = 32: its block 0; block 1 may still be on its way) and its phase factors and queries are in LDS,
        // and everyone is done with what the next sends overwrite
        if (M == 16 || sl == s_begin) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)" ::: "memory");
        bare_barrier();
        // an opaque copy per slice: the gather addresses made from these must not be hoisted out of the slice loop (they would
        // take several registers per pass)
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j) asm volatile("" : "+v"(ccall[p][i][j]));
        const unsigned slot_sel = M == 16 ? (unsigned)(2 + buf) << 16 : 0u;
        auto issue = [&](int p, int st) {
            const int blk = st / 4;
            const unsigned psel = (0x0c000000u | (unsigned)(4 + st % 4) << 8) | (M == 16 ? slot_sel : (unsigned)(2 + blk) << 16);
#pragma unroll
            for (int ab = 0; ab < 2; ++ab)
                v[(p * NST + st) % NBUF][ab] = lds_read_b128(__builtin_amdgcn_perm(ccall[p][ab][blk], xreg[st % 4], psel));
        };
        // q' = q conj(E_lo) for the pair of passes k (Re(conj(q) a E_hi E_lo) = Re(conj(q') a E_hi))
        // HALF: for pass k, the lane's 4 elements
        auto fold = [&](int k) __attribute__((always_inline)) {
            const int ln = fresh_lane(), odd = ln >> 4 & 1;
            unsigned lo = aux0 + (at0 & 0xffffu);
            if constexpr (HALF) {
                if (k > 0) lo = aux0 + (unsigned)(((qd[k] - 4 * wave - (ln >> 2 & 3)) & (kLo - 1)) + odd * kLo) * 16u;
                const uint4_t e = lds_read_b128(lo);
                const int h = ln & 3;
                const unsigned at = aux0 + (unsigned)(kAuxQ + (k * G + h) * (a.q_bf16 ? 1 : 2)) * 16u + odd * (a.q_bf16 ? 8u : 16u);
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
            if (k > 0) {
                const int d0 = qd[2 * k % NP], d1 = qd[2 * k + 1 < NP ? 2 * k + 1 : 2 * k % NP], D = odd ? d1 : d0;
                lo = aux0 + (unsigned)((D - 4 * wave - (ln >> 2 & 3)) & (kLo - 1)) * 16u;
            }
            const uint4_t e0 = lds_read_b128(lo), e1 = lds_read_b128(lo + kLo * 16u);
#pragma unroll
            for (int x = 0; x < NGRP; ++x) {
                const int h = 4 * x + (ln & 3);
                const unsigned at = aux0 + (unsigned)(kAuxQ + ((2 * k + odd) * G + h) * (a.q_bf16 ? 1 : 2)) * 16u;
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
        // the lane's place among the coarse factors of a pass whose first token is D away from its query
        auto hi_row = [&](int D) {
            const int ln = fresh_lane();
            const int row = ((D - 4 * wave - (ln >> 2 & 3)) >> kLoBits) - ((D + 1) >> kLoBits) + 8 - (ln & 3) - 4 * (ln >> 5);
            ehi_at = aux0 + (unsigned)(kAuxHi + 2 * row + (ln >> 4 & 1)) * 16u;
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
            if (p == 0) ehi_at = aux0 + (at0 >> 16);
            else if (__builtin_expect(chg >> p & 1u, 0)) hi_row(qd[p]);
            eh = lds_read_b128(ehi_at + (unsigned)(p * 2 * kHiRows * 16));
            // What the next slice needs sets out spread over this one's passes (a burst of sends fills the memory pipe's queue and
            // stops the wavefronts): its codebook (M = 16; two blocks' are sent at the end of the last pass), phase factors and queries
            if (more) {
                if (M == 16) {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (p == j * (NP - 1) / 5) send_part(sl + 1, 0, buf ^ 1, j);
                }
                if (p == (M == 16 ? 4 * (NP - 1) / 5 : (NP - 1) / 3)) send_aux(sl + 1, buf ^ 1);
            }
            // (cleared by a small matrix instruction: the compiler makes five moves of a vector of zeros)
            acc = __builtin_amdgcn_mfma_f32_4x4x1f32(zero, zero, floatx4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
            for (int st = 0; st < NST; ++st) {
                const uint4_t pa = v[(p * NST + st) % NBUF][0], pb2 = v[(p * NST + st) % NBUF][1];
                const uint8v_t both = {pa[0], pa[1], pa[2], pa[3], pb2[0], pb2[1], pb2[2], pb2[3]};
                acc = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(selv, __builtin_bit_cast(bf16x16_t, both), acc, (int)sidx, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (M == 32 && p == 0 && st + NBUF == 4) {
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // block 1 of this slice has arrived
                    bare_barrier();
                }
                if (st + NBUF < NST) issue(p, st + NBUF);
                else if (p + 1 < NP) issue(p + 1 < NP ? p + 1 : p, st + NBUF - NST);  // (after the last pass: of codes 0, not used)
                __builtin_amdgcn_sched_barrier(0);
                if (M == 32 && p == NP - 1 && st == 3 && more) {
                    // everyone has read the last pieces of block 0: the next slice's may come
                    bare_barrier();
                    send_block(sl + 1, 0, 0);
                }
                if (M == 32 && p == NP - 1 && st == 7 && more) {
                    bare_barrier();
                    send_block(sl + 1, 1, 1);
                }
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

    // Write-out.  A wavefront's tokens are scattered over the pass (4 fine positions x 8 coarse rows), so the logits of
    // four heads at a time are transposed through the now idle codebook blocks, [head][pass][coarse row][68] floats (rows
    // padded from 64: the 64 lanes of a write fall on 64 different banks), and leave as runs of 256 consecutive tokens
    // per wavefront, whose (max, sum of exp) are taken on the way.  A slice group leaves partial logits in its own array;
    // the statistics then come from k_score_combine.
    float *stg = reinterpret_cast<float *>(tab);
    float2 *wst = reinterpret_cast<float2 *>(reinterpret_cast<char *>(tab) + kWstOff);
    const int4 *segs = reinterpret_cast<const int4 *>(reinterpret_cast<const char *>(tab) + kSegOff);
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

#include "commvq_pairs.hpp"

// ------------------------------------------------------------------ k_score_combine
// Score tiles that were also cut along the codebook slices (short contexts): the logit of a token is the sum of the
// partial logits of the slice groups (Eq. new_attention's sum over the sub-spaces, split in `groups` parts).  One
// workgroup per (sequence, query head, 1024 tokens): adds the parts in a fixed order, writes the logits (over the
// first group's part) and the (max, sum of exp) of its 1024 tokens.
// Bound by latency: all parts of all its tokens are requested at once.  (A branch per part and a round of
// requests per 256 tokens went through 4 KB of instructions that had to be fetched on the way: whole calls in microseconds, so -> now, paired keys
// R = 11: two KV heads of one 400 tokens 18.8 -> 17.7, 2000 20.1 -> 17.7, 8 x 4 heads 400 20.3 -> 19.2, 1000 21.8 -> 19.7, R = 21 4000 25.4 -> 24.6;
// 32 codebooks, 8 x 4 heads 8000 27.6 -> 26.9, 32768 50.8 -> 50.6.)  Part by part of the tokens, and none past the row: the parts one after the other, with
// reads past the row that return zero, took 5.95 us for one sequence of 17107 tokens, 8 x 8 heads in four groups (5.6 so), 5.58 for 24 of 600 (5.08).
constexpr int kCombineThreads = 256, kCombineTokens = 1024;
template <int GROUPS>
__global__ __launch_bounds__(kCombineThreads) void k_score_combine(float *scores, float2 *__restrict__ sstat, const int32_t *__restrict__ cu,
                                                                  int Hq, int nsplit, long long part_stride)
{
    __shared__ float red[kCombineThreads / 64];
    int id = blockIdx.x;
    const int tile = id % nsplit;
    id /= nsplit;
    const int h = id % Hq, b = id / Hq;
    const int cu0 = cu[b], L = cu[b + 1] - cu0;
    const int t0 = tile * kCombineTokens;
    if (t0 >= L) return;
    float *const row = scores + (size_t)cu0 * Hq + (size_t)h * L;
    constexpr int MAXV = kCombineTokens / kCombineThreads;
    float part[MAXV][GROUPS];
#pragma unroll
    for (int k = 0; k < MAXV; ++k) {
        const int tok = t0 + k * kCombineThreads + (int)threadIdx.x;
#pragma unroll
        for (int e = 0; e < GROUPS; ++e) part[k][e] = tok < L ? row[(size_t)e * part_stride + (unsigned)tok] : 0.f;
    }
    __builtin_amdgcn_sched_barrier(0);
    float v[MAXV], mx = -INFINITY;
    const __amdgpu_buffer_rsrc_t own = make_rsrc(row, (unsigned)L * 4u);
#pragma unroll
    for (int k = 0; k < MAXV; ++k) {                          // in a fixed order, over the first group's part
        const int tok = t0 + k * kCombineThreads + (int)threadIdx.x;
        float acc = part[k][0];
#pragma unroll
        for (int e = 1; e < GROUPS; ++e) acc += part[k][e];
        v[k] = tok < L ? acc : -INFINITY;
        mx = fmaxf(mx, v[k]);
        if (tok < L) store_through(acc, own, (unsigned)tok * 4u);
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    mx = wave_max(mx);
    if (lane == 0) red[wave] = mx;
    __syncthreads();
    {
        float m2 = red[0];
        for (int w = 1; w < kCombineThreads / 64; ++w) m2 = fmaxf(m2, red[w]);
        mx = m2;
    }
    __syncthreads();
    float l = 0.f;
#pragma unroll
    for (int k = 0; k < MAXV; ++k)
        if (v[k] != -INFINITY) l += __builtin_amdgcn_exp2f((v[k] - mx) * kLog2e);
    l = wave_sum(l);
    if (lane == 0) red[wave] = l;
    __syncthreads();
    if (threadIdx.x == 0) {
        float lt = 0.f;
        for (int w = 0; w < kCombineThreads / 64; ++w) lt += red[w];  // fixed order
        sstat[((size_t)b * Hq + h) * nsplit + tile] = make_float2(mx, lt);
    }
}

// ------------------------------------------------------------------ position-free keys: scalar look-up table
// The case the paper sets aside in Sec. 4.2: if the rotation did not depend on the token (keys quantized
// after RoPE, or no positional rotation at all), (q C^T) could be computed once and every token's
// score would be M scalar look-ups:  s_i = sum_m T[m][code_i,m],  T[m][c] = scale * q . C[m][c].
//
// k_lut_build: T[b][g][m][c][G] fp32 (G < 4; for G >= 4 in the LDS-image order of k_score_lut, see below), one thread
// per (b, g, m, c) row; the G queries sit in LDS.
template <int G, bool BF16>
__global__ __launch_bounds__(256) void k_lut_build(const void *__restrict__ q, const void *__restrict__ cb,
                                                   float *__restrict__ lut, int Hkv, int M, int q_bf16, float scale)
{
    __shared__ float qs[G][kD];
    const int rows_per_head = M * kK;                       // rows of one KV head
    const int blocks_per_head = rows_per_head / 256;
    const int bg = blockIdx.x / blocks_per_head;            // b * Hkv + g
    const int g = bg % Hkv, b = bg / Hkv;
    const int row = (blockIdx.x % blocks_per_head) * 256 + threadIdx.x;  // m * K + c
    for (int x = threadIdx.x; x < G * kD; x += 256) {
        const size_t i = ((size_t)b * Hkv * G + (size_t)g * G) * kD + x;
        const float v = q_bf16 ? __builtin_bit_cast(float, (unsigned)static_cast<const uint16_t *>(q)[i] << 16)
                               : static_cast<const float *>(q)[i];
        qs[x / kD][x % kD] = v * scale;
    }
    __syncthreads();
    float acc[G];
#pragma unroll
    for (int h = 0; h < G; ++h) acc[h] = 0.f;
    const size_t base = ((size_t)g * rows_per_head + row) * kD;
#pragma unroll 8
    for (int e = 0; e < kD; ++e) {
        const float v = cb_elem<BF16>(cb, base + e);
#pragma unroll
        for (int h = 0; h < G; ++h) acc[h] = __builtin_fmaf(qs[h][e], v, acc[h]);
    }
    if (G >= 4) {
        // groups of four heads: the table leaves in the order k_score_lut keeps it in LDS, [b][g][head group][block of 16
        // codebooks][codeword][codebook of the block][4 heads] -- one 16-byte bank column per codebook
        const int m = row / kK, c = row % kK;
#pragma unroll
        for (int grp = 0; grp < G / 4; ++grp) {
            float4 *dst = reinterpret_cast<float4 *>(lut) +
                          (((size_t)bg * (G / 4) + grp) * (M / 16) + m / 16) * (kK * 16) + (size_t)c * 16 + (m & 15);
            *dst = make_float4(acc[(4 * grp + 0) % G], acc[(4 * grp + 1) % G], acc[(4 * grp + 2) % G], acc[(4 * grp + 3) % G]);
        }
    } else {
        float *dst = lut + ((size_t)bg * rows_per_head + row) * G;
#pragma unroll
        for (int h = 0; h < G; ++h) dst[h] = acc[h];
    }
}

// k_lut_build_mfma: the same table for bf16 codebooks and four or eight heads per KV head, where T = scale q C^T is the
// one dense (heads x M K x d) contraction of these paths: a wavefront takes 16 codebook rows, v_mfma_f32_16x16x32_bf16 with
// the queries as first operand (row = head; a bf16 query as it is, an fp32 query split exactly into three bf16 parts)
// and 16 bytes of a codebook row per lane as second.  Result lane (n, rg) holds heads 4 rg .. 4 rg + 3 of row n: one
// 16-byte entry of head group rg, stored in the LDS-image order of k_score_lut.
template <int G>
__global__ __launch_bounds__(256) void k_lut_build_mfma(const void *__restrict__ q, const uint16_t *__restrict__ cb,
                                                        float *__restrict__ lut, int Hkv, int M, int q_bf16, float scale)
{
    const int rows_per_head = M * kK;
    const int blocks_per_head = rows_per_head / 64;          // 4 wavefronts x 16 rows per workgroup
    const int bg = blockIdx.x / blocks_per_head;             // b * Hkv + g
    const int g = bg % Hkv;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane & 15, kg = lane >> 4;
    const int row = (blockIdx.x % blocks_per_head) * 64 + 16 * wave + n;  // m * K + c
    floatx4_t acc = {0.f, 0.f, 0.f, 0.f};
    const uint16_t *crow = cb + ((size_t)g * rows_per_head + row) * kD + 8 * kg;
    const size_t qbase = ((size_t)bg * G + (size_t)n) * kD + 8 * kg;  // head n of the group (rows G .. 15: zero)
#pragma unroll
    for (int ks = 0; ks < kD / 32; ++ks) {
        const uint4 B = *reinterpret_cast<const uint4 *>(crow + 32 * ks);
        if (q_bf16) {
            uint4 A = make_uint4(0u, 0u, 0u, 0u);
            if (n < G) A = *reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(q) + qbase + 32 * ks);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, A), __builtin_bit_cast(bf16x8_t, B), acc, 0, 0, 0);
        } else {
            float qf[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) qf[e] = n < G ? static_cast<const float *>(q)[qbase + 32 * ks + e] : 0.f;
            unsigned part[3][4];
#pragma unroll
            for (int e = 0; e < 8; ++e) {  // top 16 bits, top 16 bits of the rest, the rest: 8 + 8 + 8 mantissa bits, exact
                const unsigned u0 = __builtin_bit_cast(unsigned, qf[e]) & 0xffff0000u;
                const float r1 = qf[e] - __builtin_bit_cast(float, u0);
                const unsigned u1 = __builtin_bit_cast(unsigned, r1) & 0xffff0000u;
                const float r2 = r1 - __builtin_bit_cast(float, u1);
                const unsigned u2 = __builtin_bit_cast(unsigned, r2) & 0xffff0000u;
                if (e & 1) { part[0][e / 2] |= u0; part[1][e / 2] |= u1; part[2][e / 2] |= u2; }
                else { part[0][e / 2] = u0 >> 16; part[1][e / 2] = u1 >> 16; part[2][e / 2] = u2 >> 16; }
            }
#pragma unroll
            for (int pc = 0; pc < 3; ++pc) {
                const uint4 A = make_uint4(part[pc][0], part[pc][1], part[pc][2], part[pc][3]);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, A), __builtin_bit_cast(bf16x8_t, B), acc, 0, 0, 0);
            }
        }
    }
    if (4 * kg < G) {
        const int m = row / kK, c = row % kK;
        float4 *dst = reinterpret_cast<float4 *>(lut) + (((size_t)bg * (G / 4) + kg) * (M / 16) + m / 16) * (kK * 16) + (size_t)c * 16 + (m & 15);
        *dst = make_float4(acc[0] * scale, acc[1] * scale, acc[2] * scale, acc[3] * scale);
    }
}

// k_score_lut: one workgroup per (sequence, KV head, group of HG = min(G, 4) heads, tile of TPT * 1024 tokens); the
// head group's table (M * 256 * HG floats) sits in LDS, a lane owns TPT tokens: M code bytes
// in, M look-ups of HG floats, HG logits out.  Bound by the code stream and the logit writes (HBM).
template <int M, int G, int TPT>
__global__ __launch_bounds__(kSliceThreads) void k_score_lut(const float *__restrict__ lut, const uint8_t *__restrict__ key_codes,
                                                             const int32_t *__restrict__ cu, float *__restrict__ scores,
                                                             float2 *__restrict__ sstat, const SliceDims a)
{
    constexpr int HG = G < 4 ? G : 4;
    constexpr int NGRP = G / HG;
    constexpr int TILE = TPT * kSliceThreads;
    constexpr int NW = kSliceThreads / 64;
    // the table at LDS address 0 (no static LDS in this kernel), the per-wavefront statistics behind it
    extern __shared__ __attribute__((aligned(16))) float tabf[];  // HG < 4: [M * 256][HG]; HG == 4: [M / 16][256][16][4]
    float2(*wstat)[HG] = reinterpret_cast<float2(*)[HG]>(tabf + M * kK * HG);  // [NW][HG]
    int id = blockIdx.x;
    const int g = id % a.Hkv;
    id /= a.Hkv;
    const int grp = id % NGRP;  // a workgroup takes one group of HG heads (eight heads: two workgroups per tile, each with its own table)
    id /= NGRP;
    const int tile = id % a.nsplit;
    const int b = id / a.nsplit;
    const int cu0 = cu[b];
    const int L = cu[b + 1] - cu0;
    const int t0 = tile * TILE;
    if (t0 >= L) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint8_t *codes = key_codes + ((size_t)cu0 * a.Hkv + (size_t)g * L) * M;
    float *srow = scores + (size_t)cu0 * a.Hq + (size_t)g * G * L;
    if (HG == 4) {  // the group's table is contiguous in memory, already in LDS order
        const float4 *src4 = reinterpret_cast<const float4 *>(lut) + (((size_t)b * a.Hkv + g) * NGRP + grp) * (M * kK);
        for (int x = tid; x < M * kK; x += kSliceThreads) reinterpret_cast<float4 *>(tabf)[x] = src4[x];
    } else {
        const float *src = lut + ((size_t)b * a.Hkv + g) * (M * kK) * G;
        for (int x = tid; x < M * kK; x += kSliceThreads)
#pragma unroll
            for (int h = 0; h < HG; ++h) tabf[x * HG + h] = src[(size_t)x * G + grp * HG + h];
    }
    __syncthreads();
    // HG == 4: every codebook of a block of 16 owns one 16-byte bank column (row = codeword), and lane l walks the
    // codebooks of a block in the order (rot + k) mod 16 with rot = l % 8 + 8 ((l / 16) % 2): the 16 lanes that a 16-byte
    // LDS read serves together then fall on 16 different columns whatever their codes (a [codebook][codeword] table
    // lets random codes collide: 12 clk per wavefront read against 6).  The token's 16 code bytes of the block are rotated
    // by rot bytes once, so that step k finds its code at byte k; xreg[k]: byte 0 = 16 x column, byte 3 = 1 (the second
    // 64 KiB block); one byte permute splices the code in as byte 1: address = 65536 block + 256 code + 16 column.
    const unsigned rot = ((unsigned)lane & 7u) + 8u * (((unsigned)lane >> 4) & 1u);
    unsigned xreg[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) xreg[k] = (((unsigned)k + rot) & 15u) * 16u | 1u << 24;
    float mx[HG], sc[TPT][HG];
#pragma unroll
    for (int h = 0; h < HG; ++h) mx[h] = -INFINITY;
    const int tfirst = t0 + tid;
#pragma unroll
    for (int k = 0; k < TPT; ++k) {
        const int tok = tfirst + k * kSliceThreads;
        const int tc = min(tok, L - 1);
        float acc[HG];
        floatx4_t accv = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int h = 0; h < HG; ++h) acc[h] = 0.f;
#pragma unroll
        for (int v = 0; v < M / 16; ++v) {  // 16 codes at a time, 8 look-ups in flight: keeps registers flat
            const uint4 c4 = reinterpret_cast<const uint4 *>(codes + (size_t)tc * M)[v];
            unsigned cw[4] = {c4.x, c4.y, c4.z, c4.w};
            if (HG == 4) {  // rotate the 16 bytes by rot: dword selects, then a byte-granular funnel shift
#pragma unroll
                for (int st = 1; st < 4; st <<= 1) {
                    unsigned t[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) t[j] = ((rot >> 2) & (unsigned)st) ? cw[(j + st) % 4] : cw[j];
#pragma unroll
                    for (int j = 0; j < 4; ++j) cw[j] = t[j];
                }
                unsigned rv[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) rv[j] = __builtin_amdgcn_alignbyte(cw[(j + 1) % 4], cw[j], rot & 3u);
#pragma unroll
                for (int j = 0; j < 4; ++j) cw[j] = rv[j];
            }
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int x = 0; x < 8; ++x) {
                    const int kk = 8 * half + x;
                    if (HG == 4) {  // one 16-byte read, added as a vector right away
                        const unsigned sel = 0x0c000000u | (unsigned)(2 + v) << 16 | (unsigned)(4 + kk % 4) << 8;
                        const unsigned addr = __builtin_amdgcn_perm(cw[kk / 4], xreg[kk], sel);
                        const uint4_t e = lds_read_b128(addr);
                        accv += __builtin_bit_cast(floatx4_t, e);
                    } else {
                        const int m = 16 * v + kk;
                        const unsigned c = (cw[kk / 4] >> (8 * (kk % 4))) & 0xffu;
                        const float *e = tabf + ((size_t)m * kK + c) * HG;
#pragma unroll
                        for (int h = 0; h < HG; ++h) acc[h] += e[h];
                    }
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (HG == 4) {
#pragma unroll
            for (int h = 0; h < HG; ++h) acc[h] = accv[h];
        }
#pragma unroll
        for (int h = 0; h < HG; ++h) {
            sc[k][h] = acc[h];
            if (tok < L) {
                store_through(acc[h], make_rsrc(srow + (size_t)(grp * HG + h) * L, (unsigned)L * 4u), (unsigned)tok * 4u);
                mx[h] = fmaxf(mx[h], acc[h]);
            }
        }
    }
#pragma unroll
    for (int h = 0; h < HG; ++h) {
        const float wm = wave_max(mx[h]);
        float l = 0.f;
#pragma unroll
        for (int k = 0; k < TPT; ++k)
            if (tfirst + k * kSliceThreads < L) l += __builtin_amdgcn_exp2f((sc[k][h] - wm) * kLog2e);
        l = wave_sum(l);
        if (lane == 0) wstat[wave][h] = make_float2(wm, l);
    }
    __syncthreads();
    if (tid < HG) {
        float m = -INFINITY;
        for (int w = 0; w < NW; ++w) m = fmaxf(m, wstat[w][tid].x);
        float l = 0.f;
        for (int w = 0; w < NW; ++w) {
            const float2 st = wstat[w][tid];
            if (st.x != -INFINITY) l += st.y * __builtin_amdgcn_exp2f((st.x - m) * kLog2e);
        }
        sstat[((size_t)b * a.Hq + (size_t)g * G + grp * HG + tid) * a.nsplit + tile] = make_float2(m, l);
    }
}

// ------------------------------------------------------------------ k_out
struct OutArgs {
    const void *val_cb;
    const int32_t *cu;
    const unsigned *bins;
    const float *vscale, *lsum;
    float *partial, *out;
    int Hq, Hkv, nvsplit, vsplit_len, nchunk, Mv;
    int batch;
    int per_split;  // partial results per value split (k_values); 0: nchunk in all
    Divisor by_hq;
};

// Second half of the binary value code (indexed values: k_values).  Bins row r of a KV head is code bit c = vbits_code_bit(r),
// whose codebook row of d elements, in [N_c][Hkv * d], is c * Hkv + g.
// Workgroup = (sequence, KV head, chunk of codebook rows): sums the chunk's bins over the
// context splits (fixed point -> fp32 with each split's unit), then multiplies them with the
// chunk's value-codebook rows (Eq. optimized_v).
// Bound by latency: bins, units and (1024 threads) codebook rows are asked for together and ahead of the sequence's length.  Launches
// of at most a workgroup per compute unit take 1024 threads, so that 128 splits' bins are one round of loads and not four: 9.8 -> 6.5 us at
// 128K tokens, whole calls of the 8B layer 128K 106.6 -> 103.4 us, 9001 tokens 43.8 -> 42.1, 2048 code bits of 36000 81.9 -> 79.4.
// Larger launches have a second workgroup to fill such a wait: 3 x 9000 tokens, 1024 bits (384 workgroups) 62.3 -> 60.5 with 256
// threads, 63.0 with 1024; 2048 bits (768) 74.0 -> 72.5, 76.5; 3 x 43000 185.7 -> 183.3, with 1024 a hundredth slower than before.
template <int G, bool BF16, int NT>
__global__ __launch_bounds__(NT) void k_out(OutArgs a)
{
    static_assert(kOutRows == 64, "a lane per row");
    constexpr int NW = NT / 64;                                     // wavefronts: each takes every NW-th split
    constexpr int HG = NT == 1024 && G >= 4 ? 4 : 1, RG = NW / HG;  // product: HG groups of heads, RG groups of rows
    constexpr int HPG = G / HG, NCR = kOutRows / RG;                // heads and codebook rows of a wavefront
    constexpr int AT = G <= 4 || NT == 1024 ? 8 : 4;                // splits whose bins are in flight
    constexpr bool EARLY = BF16 && NT == 1024;                      // codebook rows asked for ahead of the bins' sums
    __shared__ float wsum[G][kOutRows];
    __shared__ float red[RG][G][kD];
    __shared__ __attribute__((aligned(16))) float part[NW][kOutRows][G];
    int id = blockIdx.x;
    const int chunk = id % a.nchunk;
    id /= a.nchunk;
    const int g = id % a.Hkv;
    const int b = id / a.Hkv;
    const int MK = a.Mv * kK;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // bins: [split][rows][G]: one contiguous run of 64 * G bins per split, the G bins of its row in one load per lane.  The splits
    // that the longest sequence has are asked for before this one's length is known.
    const unsigned *src = a.bins + (size_t)(b * a.Hkv + g) * a.nvsplit * G * MK + (size_t)(chunk * kOutRows + lane) * G;
    const float *units = a.vscale + ((size_t)b * a.Hq + (size_t)g * G + lane % G) * a.nvsplit;
    unsigned bv[AT][G];
    float unit = 0.f;                                               // lane k G + h: of head h in the k-th of the splits
    auto request = [&](int v0) __attribute__((always_inline)) {
        unit = units[min(v0 + lane / G % AT * NW, a.nvsplit - 1)];
#pragma unroll
        for (int k = 0; k < AT; ++k) {
            if (v0 + k * NW >= a.nvsplit) break;
            const unsigned *pv = src + (size_t)(v0 + k * NW) * G * MK;
            if (G >= 4) {
#pragma unroll
                for (int q4 = 0; q4 < G / 4; ++q4) {
                    const uint4 t4 = reinterpret_cast<const uint4 *>(pv)[q4];
                    bv[k][4 * q4] = t4.x; bv[k][(4 * q4 + 1) % G] = t4.y; bv[k][(4 * q4 + 2) % G] = t4.z; bv[k][(4 * q4 + 3) % G] = t4.w;
                }
            } else if (G == 2) {
                const uint2 t2 = *reinterpret_cast<const uint2 *>(pv);
                bv[k][0] = t2.x; bv[k][G - 1] = t2.y;
            } else {
                bv[k][0] = pv[0];
            }
        }
    };
    const int rg = wave % RG, hg = wave / RG;
    auto load_row = [&](int i) __attribute__((always_inline)) -> float2 {
        const size_t row = (size_t)vbits_code_bit(chunk * kOutRows + rg * NCR + i) * a.Hkv + g;
        if (BF16) {
            const unsigned v = static_cast<const unsigned *>(a.val_cb)[row * kJ + lane];
            return make_float2(__builtin_bit_cast(float, v), 0.f);
        }
        return static_cast<const float2 *>(a.val_cb)[row * kJ + lane];
    };
    request(wave);
    float2 rows[NCR];
    if (EARLY) {
#pragma unroll
        for (int i = 0; i < NCR; ++i) rows[i] = load_row(i);
    }
    __builtin_amdgcn_sched_barrier(0);
    const int L = a.cu[b + 1] - a.cu[b];
    const int nvs = min((L + a.vsplit_len - 1) / a.vsplit_len, a.nvsplit);
    float s[G];
#pragma unroll
    for (int hh = 0; hh < G; ++hh) s[hh] = 0.f;
    for (int v = wave; v < nvs; v += AT * NW) {
        if (v != wave) request(v);
#pragma unroll
        for (int k = 0; k < AT; ++k) {
            if (v + k * NW >= nvs) break;
#pragma unroll
            for (int hh = 0; hh < G; ++hh)
                s[hh] += (float)bv[k][hh] * __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, unit), k * G + hh));
        }
    }
#pragma unroll
    for (int hh = 0; hh < G; ++hh) part[wave][lane][hh] = s[hh];
    __syncthreads();
    for (int x = tid; x < G * kOutRows; x += NT) {
        const int hh = x % G, r = x / G;
        float t = 0.f;
#pragma unroll
        for (int q = 0; q < NW; ++q) t += part[q][r][hh];
        wsum[hh][r] = t;
    }
    __syncthreads();
    // (the wavefront's row loads are requested together)
    if (!EARLY) {
#pragma unroll
        for (int i = 0; i < NCR; ++i) rows[i] = load_row(i);
    }
    float2 acc[HPG];
#pragma unroll
    for (int hh = 0; hh < HPG; ++hh) acc[hh] = make_float2(0.f, 0.f);
#pragma unroll
    for (int i = 0; i < NCR; ++i) {
        const unsigned u = __builtin_bit_cast(unsigned, rows[i].x);
        const float2 c = BF16 ? make_float2(bf16_lo(u), bf16_hi(u)) : rows[i];
#pragma unroll
        for (int hh = 0; hh < HPG; ++hh) {
            const float w = wsum[hg * HPG + hh][rg * NCR + i];
            acc[hh].x += w * c.x;
            acc[hh].y += w * c.y;
        }
    }
#pragma unroll
    for (int hh = 0; hh < HPG; ++hh) *reinterpret_cast<float2 *>(&red[rg][hg * HPG + hh][2 * lane]) = acc[hh];
    __syncthreads();
    for (int x = tid; x < G * kD; x += NT) {
        const int hh = x / kD, e = x % kD;
        float t = 0.f;
#pragma unroll
        for (int w = 0; w < RG; ++w) t += red[w][hh][e];
        a.partial[(((size_t)b * a.Hq + (size_t)g * G + hh) * a.nchunk + chunk) * kD + e] = t;
    }
}

// Value codebook of the binary code re-laid for k_out_mfma: vp[g][kt][dim][32] bf16, where row 32 kt + j of head g is code bit
// vbits_code_bit(32 kt + j) (the row order of the bins) -- the 32 rows of a k-step of the matrix
// instruction contiguous per output dimension.  One thread per 16-byte piece of the output (static data, done once).
__global__ __launch_bounds__(256) void k_prep_values(const uint16_t *__restrict__ val_cb, uint4 *__restrict__ vp, int Hkv, int Mv)
{
    const int MK = Mv * kK;
    const size_t n = (size_t)Hkv * (MK / 32) * kD * 4;
    const size_t t = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= n) return;
    const int kg = (int)(t & 3), dim = (int)((t >> 2) % kD);
    const size_t rest = (t >> 2) / kD;
    const int kt = (int)(rest % (MK / 32)), g = (int)(rest / (MK / 32));
    unsigned w[4];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int r = 32 * kt + 8 * kg + e;
        const unsigned v = val_cb[((size_t)vbits_code_bit(r) * Hkv + g) * kD + dim];
        if (e & 1) w[e / 2] |= v << 16; else w[e / 2] = v;
    }
    vp[t] = make_uint4(w[0], w[1], w[2], w[3]);
}

// The output stage for batches (Eq. optimized_v's bins x C_V as what it is for several sequences, a matrix product):
// per KV head, [sequences x query heads] x [M_v K rows] times [rows] x [d].  A workgroup takes 16 output rows
// (16 / G sequences), kOutMfmaRows codebook rows and all d columns: it sums the fixed-point bins of its rows over the
// value splits (fp32, each split's unit applied), splits every fp32 weight EXACTLY into three bf16 parts (24 mantissa
// bits = 8 + 8 + 8) and multiplies them with the bf16 codebook by v_mfma_f32_16x16x32_bf16, accumulating in fp32: the
// fp32 product up to summation order, at a tenth of the vector instructions.  Each wavefront takes 32 of the 128 columns;
// the codebook comes straight from memory in the k_prep_values order (16 bytes per lane = 8 consecutive rows of one
// column), read once per 16 output rows instead of once per sequence.
template <int G>
__global__ __launch_bounds__(kOutThreads) void k_out_mfma(OutArgs a, const uint4 *__restrict__ vp)
{
    constexpr int KC = kOutMfmaRows, SPT = 16 / G, WS = KC + 8;  // (row stride padded: the 16 rows fall on different banks)
    __shared__ __attribute__((aligned(16))) uint16_t Wl[3][16][WS];
    int id = blockIdx.x;
    const int chunk = id % a.nchunk;  // of kOutMfmaRows rows
    id /= a.nchunk;
    const int g = id % a.Hkv;
    const int b0 = (id / a.Hkv) * SPT;
    const int MK = a.Mv * kK;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // first operand: lane (i = lane % 16, kg = lane / 16) supplies weights of output row i for rows 8 kg .. 8 kg + 7 of the
    // k-step; second: lane (n, kg) the same rows of column n; result: lane (n, rg) holds rows 4 rg .. 4 rg + 3 of column n
    const int n = lane & 15, kg = lane >> 4;
    // hi = the top 16 bits, mid = the top 16 bits of what is left, lo = the rest (exact: 8 + 8 + 8 mantissa bits)
    auto put = [&](int sq, int k, const float (&w)[G]) {
#pragma unroll
        for (int hh = 0; hh < G; ++hh) {
            const unsigned u0 = __builtin_bit_cast(unsigned, w[hh]) & 0xffff0000u;
            const float r1 = w[hh] - __builtin_bit_cast(float, u0);
            const unsigned u1 = __builtin_bit_cast(unsigned, r1) & 0xffff0000u;
            const float r2 = r1 - __builtin_bit_cast(float, u1);
            const unsigned u2 = __builtin_bit_cast(unsigned, r2) & 0xffff0000u;
            Wl[0][sq * G + hh][k] = (uint16_t)(u0 >> 16);
            Wl[1][sq * G + hh][k] = (uint16_t)(u1 >> 16);
            Wl[2][sq * G + hh][k] = (uint16_t)(u2 >> 16);
        }
    };
    auto load_bins = [](const unsigned *pv, unsigned (&bv)[G]) {
        if constexpr (G >= 4) {
#pragma unroll
            for (int q4 = 0; q4 < G / 4; ++q4) {
                const uint4 t4 = reinterpret_cast<const uint4 *>(pv)[q4];
                bv[4 * q4] = t4.x; bv[4 * q4 + 1] = t4.y; bv[4 * q4 + 2] = t4.z; bv[4 * q4 + 3] = t4.w;
            }
        } else if constexpr (G == 2) {
            const uint2 t2 = *reinterpret_cast<const uint2 *>(pv);
            bv[0] = t2.x; bv[1] = t2.y;
        } else {
            bv[0] = pv[0];
        }
    };
    if (a.nvsplit == 1) {
        // one value split: a thread's bins of all SPT sequences travel together.  Whole call with the form below and with this one, inputs
        // changing from pass to pass: 64 sequences of 512..1024 tokens, 4096 bits 109.3 -> 107.8 us, 130 of them 241.2 -> 238.2, 260 of
        // 64..128, 1024 bits 183.2 -> 180.7
        static_assert(KC == kOutThreads, "a thread takes one codebook row of every sequence");
        unsigned bv[SPT][G];
        float unit[SPT][G];
#pragma unroll
        for (int i = 0; i < SPT; ++i) {
#pragma unroll
            for (int hh = 0; hh < G; ++hh) { bv[i][hh] = 0u; unit[i][hh] = 0.f; }
            const int b = b0 + i;
            if (b < a.batch && a.cu[b + 1] > a.cu[b]) {
                load_bins(a.bins + (size_t)(b * a.Hkv + g) * G * MK + (size_t)(chunk * KC + tid) * G, bv[i]);
#pragma unroll
                for (int hh = 0; hh < G; ++hh) unit[i][hh] = a.vscale[(size_t)b * a.Hq + (size_t)g * G + hh];
            }
        }
#pragma unroll
        for (int i = 0; i < SPT; ++i) {
            float w[G];
#pragma unroll
            for (int hh = 0; hh < G; ++hh) w[hh] = (float)bv[i][hh] * unit[i][hh];
            put(i, tid, w);
        }
    } else {
        for (int it = tid; it < SPT * KC; it += kOutThreads) {
            const int sq = it / KC, k = it % KC, b = b0 + sq;
            float w[G];
#pragma unroll
            for (int hh = 0; hh < G; ++hh) w[hh] = 0.f;
            if (b < a.batch) {
                const int L = a.cu[b + 1] - a.cu[b];
                const int nvs = min((L + a.vsplit_len - 1) / a.vsplit_len, a.nvsplit);
                const unsigned *src = a.bins + (size_t)(b * a.Hkv + g) * a.nvsplit * G * MK + (size_t)(chunk * KC + k) * G;
                const float *scl = a.vscale + ((size_t)b * a.Hq + (size_t)g * G) * a.nvsplit;
#pragma unroll 4
                for (int v = 0; v < nvs; ++v) {
                    unsigned bv[G];
                    load_bins(src + (size_t)v * G * MK, bv);
#pragma unroll
                    for (int hh = 0; hh < G; ++hh) w[hh] += (float)bv[hh] * scl[(size_t)hh * a.nvsplit + v];
                }
            }
            put(sq, k, w);
        }
    }
    __syncthreads();
    floatx4_t acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    const uint4 *bsrc = vp + (((size_t)g * (MK / 32) + (size_t)chunk * (KC / 32)) * kD + 32 * wave + n) * 4 + kg;
#pragma unroll
    for (int kt = 0; kt < KC / 32; ++kt) {
        const uint4 B0 = bsrc[(size_t)(kt * kD) * 4], B1 = bsrc[(size_t)(kt * kD + 16) * 4];
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            const uint4 A = *reinterpret_cast<const uint4 *>(&Wl[p][n][32 * kt + 8 * kg]);
            acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, A), __builtin_bit_cast(bf16x8_t, B0), acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, A), __builtin_bit_cast(bf16x8_t, B1), acc[1], 0, 0, 0);
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = 4 * kg + r, b = b0 + i / G, hh = i % G;
        if (b < a.batch) {
            float *dst = a.partial + (((size_t)b * a.Hq + (size_t)g * G + hh) * a.nchunk + chunk) * kD + 32 * wave + n;
            dst[0] = acc[0][r];
            dst[16] = acc[1][r];
        }
    }
}

// One workgroup per (sequence, head): sum of the chunk partials in a fixed order, division
// by the softmax denominator (sum of the value splits' exp-sums).  Four threads per output element take every
// fourth chunk each, so that a thread's loads are one round of independent requests; their four sums are then
// added in a fixed order.  Measured: finishing inside k_out by a last-arriving workgroup costs more than this
// launch, because the device-scope release/acquire it needs writes back and invalidates L2.
// AHEAD: rows that a thread asks for before it knows the sequence's length, as many as the longest sequence has for it, up to 16: with four at
// least, batches of short sequences went through the same row several times.  4096 workgroups with 4 rows each 9.3 -> 6.2 us, 16384
// 31.2 -> 19.2, 8192 with 16 rows 16.5 -> 12.3; whole calls, 64 sequences of 100 tokens, 8 x 8 heads 93.3 -> 89.9.
constexpr int kFinalParts = 4;
template <int AHEAD>
__global__ __launch_bounds__(kD * kFinalParts) void k_out_final(OutArgs a)
{
    __shared__ float l_s;
    __shared__ float part[kFinalParts][kD];
    const int bh = blockIdx.x;
    const int b = quotient(bh, a.by_hq);
    const int e = threadIdx.x % kD, q = __builtin_amdgcn_readfirstlane(threadIdx.x / kD);
    const int rows = a.per_split ? a.nvsplit * a.per_split : a.nchunk;
    const float *pp = a.partial + (size_t)bh * rows * kD + e, *lp = a.lsum + (size_t)bh * a.nvsplit;
    // What the longest sequence has of exp-sums and of the first partial results is asked for before this sequence's length is known:
    // that, they and they again one after the other are 0.8 us.
    const float l0 = (int)threadIdx.x < min(a.nvsplit, 64) ? lp[threadIdx.x] : 0.f;
    float ahead[AHEAD];
#pragma unroll
    for (int i = 0; i < AHEAD; i += 4)
        if (i == 0 || q + i * kFinalParts < rows) {
#pragma unroll
            for (int k = i; k < i + 4 && k < AHEAD; ++k) ahead[k] = pp[(size_t)min(q + k * kFinalParts, rows - 1) * kD];
        }
    __builtin_amdgcn_sched_barrier(0);
    const int L = a.cu[b + 1] - a.cu[b];
    const int nvs = min((L + a.vsplit_len - 1) / a.vsplit_len, a.nvsplit);
    const int n = a.per_split ? nvs * a.per_split : a.nchunk;
    if (threadIdx.x < 64) {
        float l = (int)threadIdx.x < nvs ? l0 : 0.f;
        for (int v = threadIdx.x + 64; v < nvs; v += 64) l += lp[v];
        l = wave_sum(l);
        if (threadIdx.x == 0) l_s = l;
    }
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < AHEAD; ++k)
        if (q + k * kFinalParts < n) s += ahead[k];
#pragma unroll 16
    for (int c = q + AHEAD * kFinalParts; c < n; c += kFinalParts) s += pp[(size_t)c * kD];
    part[q][e] = s;
    __syncthreads();
    if (q == 0) {
        float t = part[0][e];
#pragma unroll
        for (int k = 1; k < kFinalParts; ++k) t += part[k][e];
        a.out[(size_t)bh * kD + e] = l_s > 0.f ? t / l_s : 0.f;  // a sequence without context tokens: zeros
    }
}

// ------------------------------------------------------------------ host side
// What can be checked of a batch shape from host values alone.
commvq_status check_shape(const commvq_handle *h, int32_t batch, int64_t total_tokens, int32_t max_seqlen, bool explicit_positions)
{
    if (batch < 1 || max_seqlen < 1) return COMMVQ_ERR_SHAPE;
    if (total_tokens < max_seqlen) return COMMVQ_ERR_SHAPE;
    if (total_tokens > (int64_t)batch * max_seqlen) return COMMVQ_ERR_SHAPE;
    if (total_tokens > (int64_t)1 << 30) return COMMVQ_ERR_SHAPE;
    // the kernels address one (sequence, KV head)'s codes and logits with 32-bit byte offsets (paired keys: the bound is that of
    // two index bytes per level of whole blocks of 16)
    const commvq_config &c = h->cfg;
    int64_t rec = bin_values(c) ? c.value_bits / 8 : c.m_val;
    if (pair_keys(c)) rec = std::max<int64_t>(rec, 32 * pair_blocks(c));
    else rec = std::max<int64_t>(rec, c.m_key);
    rec = std::max<int64_t>(rec, 4 * h->G);
    if ((int64_t)max_seqlen * rec > (int64_t)0xffffffffll) return COMMVQ_ERR_SHAPE;
    // keys at positions 0 .. L - 1 and the query at or after the last of them: the farthest key is at least
    // max_seqlen - 1 away, which the phase tables must cover (Eq. rope_ri is exact only inside them)
    if (!explicit_positions && !c.position_free && (int64_t)max_seqlen - 1 > c.max_position) return COMMVQ_ERR_SHAPE;
    return COMMVQ_OK;
}

commvq_status check_positions(const commvq_handle *h, const commvq_positions *p)
{
    if (!p) return COMMVQ_ERR_NULL;
    if (!p->cu_seqlens || !p->q_pos) return COMMVQ_ERR_NULL;
    return check_shape(h, p->batch, p->total_tokens, p->max_seqlen, p->key_pos != nullptr);
}

commvq_status prep(const commvq_handle *h, const commvq_positions *pos, void *workspace, size_t workspace_bytes,
                   Plan *plan, Workspace *w)
{
    if (!h) return COMMVQ_ERR_NULL;
    commvq_status st = check_positions(h, pos);
    if (st != COMMVQ_OK) return st;
    if (pair_keys(h->cfg) && pos->key_pos) return COMMVQ_ERR_CONFIG;  // paired-code keys: contiguous positions only
    make_plan(h, pos->batch, pos->total_tokens, pos->max_seqlen, use_sliced(h, pos->key_pos != nullptr), plan);
    carve(h, pos->batch, pos->total_tokens, pos->max_seqlen, workspace, w);
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) || workspace_bytes < w->bytes)
        return COMMVQ_ERR_WORKSPACE;
    if (h->device < 0) return COMMVQ_ERR_NO_DEVICE;  // planner handle: every argument was acceptable, nothing is launched
    return COMMVQ_OK;
}

struct ScoreArgs {
    const void *q;
    const uint8_t *key_codes;
    const void *key_cb;
    const int32_t *cu, *q_pos, *key_pos;
    const float2 *tbl_hi, *tbl_lo;
    float *scores;
    float2 *sstat;
    ScoreDims d;
};

// Tiles of 16 tokens go to k_score_few (there are then fewer than 2 kScoreMinWgs of them: each dimension of its grid is in range), except
// fp32 rows of 32 codebooks with 4 or 8 heads, where it takes 256 registers, one wavefront per SIMD, which pays only while there is
// about one workgroup per SIMD.  Whole calls in microseconds, k_score against it: 4 heads, 656 workgroups 28.5 and 28.1, 800 31.0 and
// 32.1, 4000 78.1 and 85.4; 8 heads, 1500 63.0 and 61.6, 2000 69.9 and 70.2, 4000 104.5 and 108.5.  (1 and 2 heads, 16 codebooks and bf16:
// faster with it by 4 to 30 % up to 4000, which one KV head reaches at 65000 tokens: one fp32 head, 32 codebooks 8000 tokens 19.4 and 17.0,
// 32000 43.4 and 37.1, 65000 75.6 and 64.3; 8 heads, 16 codebooks 65000 89.2 and 69.3; explicit positions, bf16, 4 heads, 16 codebooks 53.7 and 41.4.)
template <int M, int G>
hipError_t launch_score_mg(const ScoreArgs &a, bool bf16, int batch, hipStream_t s)
{
    const bool wide = !bf16 && M == 32 && G >= 4;
    const bool few = a.d.split_len == kFewTokens && (!wide || batch * a.d.Hkv * a.d.nsplit <= (G == 4 ? 700 : 1800));
    auto kernel = few ? (bf16 ? k_score_few<M, G, true> : k_score_few<M, G, false>) : (bf16 ? k_score<M, G, true> : k_score<M, G, false>);
    const dim3 grid = few ? dim3(a.d.Hkv, a.d.nsplit, batch) : dim3(batch * a.d.Hkv * a.d.nsplit);
    hipLaunchKernelGGL(kernel, grid, dim3(kScoreThreads), 0, s, a.q, a.key_codes, a.key_cb, a.cu, a.q_pos, a.key_pos, a.tbl_hi,
                       a.tbl_lo, a.scores, a.sstat, a.d);
    return hipGetLastError();
}
template <int M>
hipError_t launch_score_m(const ScoreArgs &a, int G, bool bf16, int batch, hipStream_t s)
{
    switch (G) {
    case 1: return launch_score_mg<M, 1>(a, bf16, batch, s);
    case 2: return launch_score_mg<M, 2>(a, bf16, batch, s);
    case 4: return launch_score_mg<M, 4>(a, bf16, batch, s);
    default: return launch_score_mg<M, 8>(a, bf16, batch, s);
    }
}

template <int G>
hipError_t launch_out_g(const OutArgs &a, bool bf16, int grid, hipStream_t s)
{
    if (grid <= 256) {
        if (bf16) hipLaunchKernelGGL((k_out<G, true, 1024>), dim3(grid), dim3(1024), 0, s, a);
        else hipLaunchKernelGGL((k_out<G, false, 1024>), dim3(grid), dim3(1024), 0, s, a);
    } else {
        if (bf16) hipLaunchKernelGGL((k_out<G, true, kOutThreads>), dim3(grid), dim3(kOutThreads), 0, s, a);
        else hipLaunchKernelGGL((k_out<G, false, kOutThreads>), dim3(grid), dim3(kOutThreads), 0, s, a);
    }
    return hipGetLastError();
}

struct StreamArgs {
    const void *q;
    const uint8_t *key_codes;
    const uint4 *packed;
    const int32_t *cu, *q_pos;
    const float2 *tbl_hi, *tbl_lo;
    float *scores;
    float2 *sstat;
    StreamDims d;
};

template <int M, int FORM, int NP>
hipError_t launch_stream_n(const StreamArgs &a, int grid, hipStream_t s)
{
    static std::atomic<uint64_t> lds_ok{0};  // per instantiation and device
    if (hipError_t e = allow_dynamic_lds(&k_score_stream<M, FORM, NP>, kStreamLds, lds_ok); e != hipSuccess) return e;
    hipLaunchKernelGGL((k_score_stream<M, FORM, NP>), dim3(grid), dim3(kSliceThreads), kStreamLds, s, a.q, a.key_codes,
                       a.packed, a.cu, a.q_pos, a.tbl_hi, a.tbl_lo, a.scores, a.sstat, a.d);
    return hipGetLastError();
}
template <int M, int FORM>
hipError_t launch_stream_g(const StreamArgs &a, int passes, int grid, hipStream_t s)
{
    switch (passes) {
    case 2: return launch_stream_n<M, FORM, 2>(a, grid, s);
    case 3: return launch_stream_n<M, FORM, 3>(a, grid, s);
    case 4: return launch_stream_n<M, FORM, 4>(a, grid, s);
    case 5: return launch_stream_n<M, FORM, 5>(a, grid, s);
    case 6: return launch_stream_n<M, FORM, 6>(a, grid, s);
    case 7: return launch_stream_n<M, FORM, 7>(a, grid, s);
    default: return launch_stream_n<M, FORM, 8>(a, grid, s);
    }
}
hipError_t launch_stream(const StreamArgs &a, int M, int passes, bool exchange, int grid, hipStream_t s)
{
    if (exchange)
        return passes == 2 ? launch_stream_n<16, 0, 2>(a, grid, s) : passes == 4 ? launch_stream_n<16, 0, 4>(a, grid, s)
             : passes == 6 ? launch_stream_n<16, 0, 6>(a, grid, s) : launch_stream_n<16, 0, 8>(a, grid, s);
    if (M == 16) return a.d.G == 8 ? launch_stream_g<16, 2>(a, passes, grid, s) : launch_stream_g<16, 1>(a, passes, grid, s);
    return a.d.G == 8 ? launch_stream_g<32, 2>(a, passes, grid, s) : launch_stream_g<32, 1>(a, passes, grid, s);
}

template <int SETS, int FORM, int NP>
hipError_t launch_pair_n(const StreamArgs &a, int R, int PB, int grid, hipStream_t s)
{
    static std::atomic<uint64_t> lds_ok{0};  // per instantiation and device
    if (hipError_t e = allow_dynamic_lds(&k_score_pair<SETS, FORM, NP>, kPairLds, lds_ok); e != hipSuccess) return e;
    hipLaunchKernelGGL((k_score_pair<SETS, FORM, NP>), dim3(grid), dim3(kSliceThreads), kPairLds, s, a.q, a.key_codes,
                       a.packed, a.cu, a.q_pos, a.tbl_hi, a.tbl_lo, a.scores, a.sstat, a.d, R, PB);
    return hipGetLastError();
}
template <int SETS>
hipError_t launch_pair_s(const StreamArgs &a, int passes, bool exchange, int R, int PB, int grid, hipStream_t s)
{
    constexpr int most = pair_passes(SETS);
    if (exchange)
        return passes == 2 ? launch_pair_n<SETS, 0, 2>(a, R, PB, grid, s) : passes == 4 ? launch_pair_n<SETS, 0, 4>(a, R, PB, grid, s)
                                                                                        : launch_pair_n<SETS, 0, most>(a, R, PB, grid, s);
    if (a.d.G == 8) {
        if (passes == 2) return launch_pair_n<SETS, 2, 2>(a, R, PB, grid, s);
        if (passes == 3) return launch_pair_n<SETS, 2, 3>(a, R, PB, grid, s);
        if (passes == 4) return launch_pair_n<SETS, 2, 4>(a, R, PB, grid, s);
        return launch_pair_n<SETS, 2, most>(a, R, PB, grid, s);
    }
    if (passes == 2) return launch_pair_n<SETS, 1, 2>(a, R, PB, grid, s);
    if (passes == 3) return launch_pair_n<SETS, 1, 3>(a, R, PB, grid, s);
    if (passes == 4) return launch_pair_n<SETS, 1, 4>(a, R, PB, grid, s);
    return launch_pair_n<SETS, 1, most>(a, R, PB, grid, s);
}
hipError_t launch_pair(const StreamArgs &a, const commvq_config &c, int passes, bool exchange, int grid, hipStream_t s)
{
    const int R = c.key_levels, PB = pair_record_bytes(c);
    switch (pair_sets(c)) {
    case 3: return launch_pair_s<3>(a, passes, exchange, R, PB, grid, s);
    case 4: return launch_pair_s<4>(a, passes, exchange, R, PB, grid, s);
    default: return launch_pair_s<6>(a, passes, exchange, R, PB, grid, s);
    }
}

// Re-lays a key codebook (index form) or a tied pair table into the LDS-image order of its score kernel.
hipError_t launch_prep(const commvq_config &c, const void *key_cb, uint4 *packed, hipStream_t s)
{
    const size_t n_pieces = packed_key_bytes(c) / 16;
    if (pair_keys(c))
        hipLaunchKernelGGL(k_prep_pairs, dim3((unsigned)((n_pieces + 255) / 256)), dim3(256), 0, s,
                           static_cast<const uint4 *>(key_cb), packed, c.n_kv_heads, c.key_levels, pair_sets(c));
    else
        hipLaunchKernelGGL(k_prep, dim3((unsigned)((n_pieces + 255) / 256)), dim3(256), 0, s,
                           static_cast<const uint4 *>(key_cb), packed, c.n_kv_heads, c.m_key);
    return hipGetLastError();
}

hipError_t launch_prep_values(const commvq_config &c, const void *val_cb, uint4 *vp, hipStream_t s)
{
    const size_t n = (size_t)c.n_kv_heads * val_books(c) * kK * kD * 2 / 16;
    hipLaunchKernelGGL(k_prep_values, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, static_cast<const uint16_t *>(val_cb), vp,
                       c.n_kv_heads, val_books(c));
    return hipGetLastError();
}

template <int M, int G, int TPT>
hipError_t launch_lut_mgt(const float *lut, const uint8_t *key_codes, const int32_t *cu, float *scores, float2 *sstat,
                          const SliceDims &d, int grid, hipStream_t s)
{
    constexpr int lds = M * kK * (G < 4 ? G : 4) * 4 + (kSliceThreads / 64) * (G < 4 ? G : 4) * 8;  // table + per-wavefront statistics
    static std::atomic<uint64_t> lds_ok{0};  // per instantiation and device
    if (hipError_t e = allow_dynamic_lds(&k_score_lut<M, G, TPT>, lds, lds_ok); e != hipSuccess) return e;
    grid *= G < 4 ? 1 : G / 4;  // one workgroup per group of four heads
    hipLaunchKernelGGL((k_score_lut<M, G, TPT>), dim3(grid), dim3(kSliceThreads), lds, s, lut, key_codes, cu, scores, sstat, d);
    return hipGetLastError();
}
template <int M, int G>
hipError_t launch_lut_mg(const void *q, const void *key_cb, bool bf16, float *lut, const uint8_t *key_codes, const int32_t *cu,
                         float *scores, float2 *sstat, const SliceDims &d, int B, int tpt, int grid, hipStream_t s)
{
    const int blocks = B * d.Hkv * (M * kK / 256);
    if (bf16 && G >= 4)  // the table as a matrix product (16 rows per wavefront, 64 per workgroup)
        hipLaunchKernelGGL((k_lut_build_mfma<G>), dim3(4 * blocks), dim3(256), 0, s, q, static_cast<const uint16_t *>(key_cb), lut, d.Hkv,
                           M, d.q_bf16, d.scale);
    else if (bf16) hipLaunchKernelGGL((k_lut_build<G, true>), dim3(blocks), dim3(256), 0, s, q, key_cb, lut, d.Hkv, M, d.q_bf16, d.scale);
    else hipLaunchKernelGGL((k_lut_build<G, false>), dim3(blocks), dim3(256), 0, s, q, key_cb, lut, d.Hkv, M, d.q_bf16, d.scale);
    if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    switch (tpt) {
    case 1: return launch_lut_mgt<M, G, 1>(lut, key_codes, cu, scores, sstat, d, grid, s);
    case 2: return launch_lut_mgt<M, G, 2>(lut, key_codes, cu, scores, sstat, d, grid, s);
    default: return launch_lut_mgt<M, G, 4>(lut, key_codes, cu, scores, sstat, d, grid, s);
    }
}
template <int M>
hipError_t launch_lut_m(int G, const void *q, const void *key_cb, bool bf16, float *lut, const uint8_t *key_codes,
                        const int32_t *cu, float *scores, float2 *sstat, const SliceDims &d, int B, int tpt, int grid, hipStream_t s)
{
    switch (G) {
    case 1: return launch_lut_mg<M, 1>(q, key_cb, bf16, lut, key_codes, cu, scores, sstat, d, B, tpt, grid, s);
    case 2: return launch_lut_mg<M, 2>(q, key_cb, bf16, lut, key_codes, cu, scores, sstat, d, B, tpt, grid, s);
    case 4: return launch_lut_mg<M, 4>(q, key_cb, bf16, lut, key_codes, cu, scores, sstat, d, B, tpt, grid, s);
    default: return launch_lut_mg<M, 8>(q, key_cb, bf16, lut, key_codes, cu, scores, sstat, d, B, tpt, grid, s);
    }
}

commvq_status run_scores(commvq_handle *h, const void *q, const uint8_t *key_codes, const void *key_cb,
                         const commvq_positions *pos, const Plan &plan, const Workspace &w, hipStream_t s)
{
    const commvq_config &c = h->cfg;
    if (c.position_free) {  // scalar look-up table: build T = scale q C^T, then M look-ups per token
        SliceDims d;
        d.Hq = c.n_q_heads; d.Hkv = c.n_kv_heads; d.nsplit = plan.score_splits; d.n_hi = h->n_hi;
        d.q_bf16 = c.q_dtype == COMMVQ_BF16; d.scale = h->scale;
        const int grid = pos->batch * c.n_kv_heads * plan.score_splits;
        const int tpt = plan.score_split_len / kSliceThreads;
        const bool bf16 = c.codebook_dtype == COMMVQ_BF16;
        hipError_t e = c.m_key == 16 ? launch_lut_m<16>(h->G, q, key_cb, bf16, w.lut, key_codes, pos->cu_seqlens, w.scores, w.sstat, d, pos->batch, tpt, grid, s)
                                     : launch_lut_m<32>(h->G, q, key_cb, bf16, w.lut, key_codes, pos->cu_seqlens, w.scores, w.sstat, d, pos->batch, tpt, grid, s);
        return e == hipSuccess ? COMMVQ_OK : COMMVQ_ERR_LAUNCH;
    }
    if (plan.score_kernel) {  // slice-streaming kernel: needs the codebook in LDS-image order
        const uint4 *packed = nullptr;
        for (const auto &e : h->packed_keys)
            if (e.first == key_cb) packed = e.second;
        if (!packed) {  // not packed ahead of time: re-lay it into the workspace on every call
            if (launch_prep(c, key_cb, w.packed, s) != hipSuccess) return COMMVQ_ERR_LAUNCH;
            packed = w.packed;
        }
        hipError_t e;
        const StreamShape &ss = plan.stream;
        StreamArgs sa;
        sa.q = q; sa.key_codes = key_codes; sa.packed = packed; sa.cu = pos->cu_seqlens; sa.q_pos = pos->q_pos;
        sa.tbl_hi = h->tbl_hi; sa.tbl_lo = h->tbl_lo; sa.scores = w.scores; sa.sstat = w.sstat;
        sa.d.Hq = c.n_q_heads; sa.d.Hkv = c.n_kv_heads; sa.d.G = h->G; sa.d.batch = pos->batch; sa.d.n_hi = h->n_hi;
        sa.d.q_bf16 = c.q_dtype == COMMVQ_BF16; sa.d.scale = h->scale;
        sa.d.tiles = ss.tiles; sa.d.groups = ss.groups;
        sa.d.nstat = stat_splits(h, plan, pos->max_seqlen);
        sa.d.part_stride = (long long)(logit_bytes(h, pos->total_tokens) / 4);
        const int grid = c.n_kv_heads * ss.tiles * ss.groups;
        const bool exchange = exchange_rows(h, ss, pos->batch, pos->total_tokens);
        e = pair_keys(c) ? launch_pair(sa, c, ss.passes, exchange, grid, s) : launch_stream(sa, c.m_key, ss.passes, exchange, grid, s);
        if (e == hipSuccess && ss.groups > 1) {
            const int ns = sa.d.nstat;
            auto combine = ss.groups == 2 ? k_score_combine<2> : ss.groups == 4 ? k_score_combine<4> : ss.groups == 8 ? k_score_combine<8> : k_score_combine<16>;
            hipLaunchKernelGGL(combine, dim3((unsigned)(pos->batch * c.n_q_heads * ns)), dim3(kCombineThreads), 0, s,
                               w.scores, w.sstat, pos->cu_seqlens, c.n_q_heads, ns, sa.d.part_stride);
            e = hipGetLastError();
        }
        return e == hipSuccess ? COMMVQ_OK : COMMVQ_ERR_LAUNCH;
    }
    ScoreArgs a;
    a.q = q; a.key_codes = key_codes; a.key_cb = key_cb;
    a.cu = pos->cu_seqlens; a.q_pos = pos->q_pos; a.key_pos = pos->key_pos;
    a.tbl_hi = h->tbl_hi; a.tbl_lo = h->tbl_lo;
    a.scores = w.scores; a.sstat = w.sstat;
    a.d.Hq = c.n_q_heads; a.d.Hkv = c.n_kv_heads; a.d.nsplit = plan.score_splits; a.d.split_len = plan.score_split_len;
    a.d.n_hi = h->n_hi; a.d.q_bf16 = c.q_dtype == COMMVQ_BF16; a.d.scale = h->scale;
    const bool bf16 = c.codebook_dtype == COMMVQ_BF16;
    hipError_t e = c.m_key == 16 ? launch_score_m<16>(a, h->G, bf16, pos->batch, s) : launch_score_m<32>(a, h->G, bf16, pos->batch, s);
    return e == hipSuccess ? COMMVQ_OK : COMMVQ_ERR_LAUNCH;
}

template <int G, int CB, int S, int NCS, int NT, bool BF16>
hipError_t launch_values_n(const ValuesArgs &a, hipStream_t s)
{
    const int lds = values_lds<G, CB, S, NCS, NT>(a.spans);
    if (a.ncg * CB != a.M || lds > kLdsBytes || (a.spans > 1 && (S > 1 || (CB == 8 && NT == 512)))) return hipErrorInvalidValue;  // (a shape that this instantiation is not for)
    static std::atomic<uint64_t> lds_ok{0};  // per instantiation and device
    if (hipError_t e = allow_dynamic_lds(&k_values<G, CB, S, NCS, NT, BF16>, kLdsBytes, lds_ok); e != hipSuccess) return e;
    const unsigned grid = (unsigned)(S == 1 ? a.batch * a.ranges : (a.batch + S - 1) / S) * (unsigned)(NCS * a.ncg * a.Hkv);
    hipLaunchKernelGGL((k_values<G, CB, S, NCS, NT, BF16>), dim3(grid), dim3(NT), lds, s, a);
    return hipGetLastError();
}
template <int G>
hipError_t launch_values_g(const ValuesArgs &a, const ValueShape &v, bool bf16, hipStream_t s)
{
    if (!bf16) return v.parts == 4 ? launch_values_n<G, 4, 1, 4, 512, false>(a, s) : launch_values_n<G, 4, 1, 1, 512, false>(a, s);
    if (v.parts == 4) return launch_values_n<G, 4, 1, 4, 512, true>(a, s);
    if constexpr (G >= 4) {
        if (v.slots == 2) return launch_values_n<G, 8, 2, 1, 512, true>(a, s);
        if constexpr (G == 4)
            if (v.slots == 4) return launch_values_n<4, 8, 4, 1, 512, true>(a, s);
        if (v.books == 8) return v.threads == 1024 ? launch_values_n<G, 8, 1, 1, 1024, true>(a, s) : launch_values_n<G, 8, 1, 1, 512, true>(a, s);
        return launch_values_n<G, 4, 1, 1, 1024, true>(a, s);
    } else {
        return launch_values_n<G, 4, 1, 1, 512, true>(a, s);
    }
}

// Value stage and product with the value codebook: mode 0 in one, 1 up to the bins, 2 from the bins on (k_values).
commvq_status run_values(commvq_handle *h, const uint8_t *val_codes, const void *val_cb, const commvq_positions *pos,
                         const Plan &plan, const Workspace &w, int mode, hipStream_t s)
{
    const commvq_config &c = h->cfg;
    ValuesArgs a;
    a.val_codes = val_codes; a.val_cb = val_cb; a.cu = pos->cu_seqlens; a.scores = w.scores; a.sstat = w.sstat;
    a.bins = w.bins; a.vscale = w.vscale; a.lsum = w.lsum; a.partial = w.partial;
    a.Hq = c.n_q_heads; a.Hkv = c.n_kv_heads; a.M = c.m_val;
    a.nsplit = stat_splits(h, plan, pos->max_seqlen); a.split_len = stat_len(h, plan);
    a.ranges = plan.values.ranges; a.range_len = plan.values.range_len; a.span = plan.values.span;
    a.spans = (a.range_len + a.span - 1) / a.span;
    a.batch = pos->batch; a.ncg = c.m_val / plan.values.books; a.mode = mode;
    a.by_hkv = divisor(a.Hkv); a.by_ncg = divisor(a.ncg); a.by_batch = divisor(a.batch); a.by_span = divisor(a.span);
    a.split_shift = __builtin_ctz(a.split_len);             // (statistics tiles are powers of two)
    hipError_t e;
    const bool bf16 = c.codebook_dtype == COMMVQ_BF16;
    switch (h->G) {
    case 1: e = launch_values_g<1>(a, plan.values, bf16, s); break;
    case 2: e = launch_values_g<2>(a, plan.values, bf16, s); break;
    case 4: e = launch_values_g<4>(a, plan.values, bf16, s); break;
    default: e = launch_values_g<8>(a, plan.values, bf16, s); break;
    }
    return e == hipSuccess ? COMMVQ_OK : COMMVQ_ERR_LAUNCH;
}

// Sum of the partial results of k_values.
void launch_out_final(const OutArgs &a, hipStream_t s)
{
    const int rows = a.per_split ? a.nvsplit * a.per_split : a.nchunk;
    auto kernel = rows <= kFinalParts ? k_out_final<1> : rows <= 4 * kFinalParts ? k_out_final<4> : k_out_final<16>;
    hipLaunchKernelGGL(kernel, dim3(a.batch * a.Hq), dim3(kD * kFinalParts), 0, s, a);
}

commvq_status run_values_final(commvq_handle *h, const commvq_positions *pos, const Plan &plan, const Workspace &w, float *out, hipStream_t s)
{
    OutArgs a = {};
    a.cu = pos->cu_seqlens; a.lsum = w.lsum; a.partial = w.partial; a.out = out;
    a.Hq = h->cfg.n_q_heads; a.Hkv = h->cfg.n_kv_heads; a.nvsplit = plan.values.ranges; a.vsplit_len = plan.values.range_len;
    a.per_split = h->cfg.m_val / plan.values.books; a.batch = pos->batch; a.by_hq = divisor(a.Hq);
    launch_out_final(a, s);
    return hipGetLastError() == hipSuccess ? COMMVQ_OK : COMMVQ_ERR_LAUNCH;
}

// Binary code: Softmax(A) S_V as an integer matrix product (commvq_vbits.hip), then its product with the codebook.
commvq_status run_bins(commvq_handle *h, const uint8_t *val_codes, const commvq_positions *pos,
                       const Plan &plan, const Workspace &w, hipStream_t s)
{
    const commvq_config &c = h->cfg;
    VbitsArgs v;
    v.val_bits = val_codes; v.cu = pos->cu_seqlens; v.scores = w.scores; v.sstat = w.sstat;
    v.bins = w.bins; v.vscale = w.vscale; v.lsum = w.lsum;
    v.Hq = c.n_q_heads; v.Hkv = c.n_kv_heads; v.G = h->G;
    v.nsplit = stat_splits(h, plan, pos->max_seqlen); v.split_len = stat_len(h, plan);
    v.nvsplit = plan.value_splits; v.vsplit_len = plan.value_split_len;
    v.Nc = c.value_bits; v.batch = pos->batch;
    return commvq_launch_vbits(v, s) == hipSuccess ? COMMVQ_OK : COMMVQ_ERR_LAUNCH;
}

commvq_status run_output(commvq_handle *h, const void *val_cb, const commvq_positions *pos, const Plan &plan,
                         const Workspace &w, float *out, hipStream_t s)
{
    const commvq_config &c = h->cfg;
    OutArgs a;
    a.val_cb = val_cb; a.cu = pos->cu_seqlens; a.bins = w.bins; a.vscale = w.vscale; a.lsum = w.lsum;
    a.partial = w.partial; a.out = out;
    a.Hq = c.n_q_heads; a.Hkv = c.n_kv_heads;
    a.nvsplit = plan.value_splits; a.vsplit_len = plan.value_split_len;
    a.nchunk = plan.out_chunks; a.Mv = val_books(c); a.batch = pos->batch; a.per_split = 0; a.by_hq = divisor(a.Hq);
    const int grid = pos->batch * c.n_kv_heads * plan.out_chunks;
    const bool bf16 = c.codebook_dtype == COMMVQ_BF16;
    hipError_t e;
    if (use_out_mfma(h, pos->batch)) {  // several sequences: the product with the value codebook on the matrix cores
        const uint4 *vp = nullptr;
        for (const auto &pv : h->packed_vals)
            if (pv.first == val_cb) vp = pv.second;
        if (!vp) {  // not packed ahead of time: re-lay the value codebook into the workspace on every call
            if (launch_prep_values(c, val_cb, w.packed_val, s) != hipSuccess) return COMMVQ_ERR_LAUNCH;
            vp = w.packed_val;
        }
        a.nchunk = val_books(c) * kK / kOutMfmaRows;
        const int spt = 16 / h->G;
        const int rows = (pos->batch + spt - 1) / spt * c.n_kv_heads;
        // A chunk per workgroup.  Two or four one after the other, for fewer partial results, made no difference of half a microsecond
        // (130 sequences of 64..128 tokens, 2048 bits 128.0 -> 127.8 us, 4096 bits 161.2 -> 160.8; of 512..1024 tokens 186.6 and 232.7 either way).
        const int mgrid = rows * a.nchunk;
        switch (h->G) {
        case 1: hipLaunchKernelGGL(k_out_mfma<1>, dim3(mgrid), dim3(kOutThreads), 0, s, a, vp); break;
        case 2: hipLaunchKernelGGL(k_out_mfma<2>, dim3(mgrid), dim3(kOutThreads), 0, s, a, vp); break;
        case 4: hipLaunchKernelGGL(k_out_mfma<4>, dim3(mgrid), dim3(kOutThreads), 0, s, a, vp); break;
        default: hipLaunchKernelGGL(k_out_mfma<8>, dim3(mgrid), dim3(kOutThreads), 0, s, a, vp); break;
        }
        if (hipGetLastError() != hipSuccess) return COMMVQ_ERR_LAUNCH;
        launch_out_final(a, s);
        return hipGetLastError() == hipSuccess ? COMMVQ_OK : COMMVQ_ERR_LAUNCH;
    }
    switch (h->G) {
    case 1: e = launch_out_g<1>(a, bf16, grid, s); break;
    case 2: e = launch_out_g<2>(a, bf16, grid, s); break;
    case 4: e = launch_out_g<4>(a, bf16, grid, s); break;
    default: e = launch_out_g<8>(a, bf16, grid, s); break;
    }
    if (e != hipSuccess) return COMMVQ_ERR_LAUNCH;
    launch_out_final(a, s);
    return hipGetLastError() == hipSuccess ? COMMVQ_OK : COMMVQ_ERR_LAUNCH;
}

}  // namespace

// ------------------------------------------------------------------ C ABI
extern "C" {

const char *commvq_status_string(commvq_status s)
{
    switch (s) {
    case COMMVQ_OK: return "ok";
    case COMMVQ_ERR_NULL: return "required pointer is NULL";
    case COMMVQ_ERR_CONFIG: return "unsupported configuration";
    case COMMVQ_ERR_SHAPE: return "inconsistent batch shape";
    case COMMVQ_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case COMMVQ_ERR_LAUNCH: return "HIP runtime error";
    case COMMVQ_ERR_NO_DEVICE: return "no usable gfx950 device";
    }
    return "unknown status";
}

commvq_status commvq_validate_config(const commvq_config *c)
{
    if (!c) return COMMVQ_ERR_NULL;
    if (c->head_dim != kD || c->k != kK) return COMMVQ_ERR_CONFIG;
    if (c->n_q_heads < 1 || c->n_kv_heads < 1 || c->n_q_heads % c->n_kv_heads) return COMMVQ_ERR_CONFIG;
    const int G = c->n_q_heads / c->n_kv_heads;
    if (G != 1 && G != 2 && G != 4 && G != 8) return COMMVQ_ERR_CONFIG;
    if (c->value_format == COMMVQ_VALUES_INDEXED) {
        if (c->m_val != 16 && c->m_val != 32) return COMMVQ_ERR_CONFIG;
    } else if (c->value_format == COMMVQ_VALUES_BINARY) {
        // towards the output kernels N_c / 256 stands in for the number of value codebooks: 4, 8 or 16
        if (c->value_bits != 1024 && c->value_bits != 2048 && c->value_bits != 4096) return COMMVQ_ERR_CONFIG;
    } else {
        return COMMVQ_ERR_CONFIG;
    }
    if (c->key_format == COMMVQ_KEYS_INDEXED) {
        if (c->m_key != 16 && c->m_key != 32) return COMMVQ_ERR_CONFIG;
    } else if (c->key_format == COMMVQ_KEYS_PAIRED) {
        // a record is at most 32 bytes (R <= 21); one table for a and b, bf16 only
        if (c->key_levels < 1 || c->key_levels > 21 || c->codebook_dtype != COMMVQ_BF16) return COMMVQ_ERR_CONFIG;
    } else {
        return COMMVQ_ERR_CONFIG;
    }
    if (c->position_free != 0 && (c->position_free != 1 || c->key_format != COMMVQ_KEYS_INDEXED)) return COMMVQ_ERR_CONFIG;
    if (c->q_dtype != COMMVQ_F32 && c->q_dtype != COMMVQ_BF16) return COMMVQ_ERR_CONFIG;
    if (c->codebook_dtype != COMMVQ_F32 && c->codebook_dtype != COMMVQ_BF16) return COMMVQ_ERR_CONFIG;
    if (!(c->rope_base > 1.0) || !(c->softmax_scale >= 0.0)) return COMMVQ_ERR_CONFIG;
    if (c->max_position < 0 || c->max_position > (1 << 24)) return COMMVQ_ERR_CONFIG;
    return COMMVQ_OK;
}

static commvq_handle *new_handle(const commvq_config *config, int device)
{
    commvq_handle *h = new (std::nothrow) commvq_handle();
    if (!h) return nullptr;
    h->cfg = *config;
    h->G = config->n_q_heads / config->n_kv_heads;
    h->scale = (float)(config->softmax_scale > 0.0 ? config->softmax_scale : 1.0 / std::sqrt((double)kD));
    // a distance ad behind the query is 64 (ad / 64) + lo, one before it -64 ceil(ad / 64) + lo, with lo on 0..63
    h->n_hi = ((config->max_position + kLo - 1) >> kLoBits) + 1;
    h->device = device;
    h->tbl_hi = h->tbl_lo = nullptr;
    h->static_scratch = nullptr;
    h->prof_every = 0; h->prof_calls = 0; h->prof_head = h->prof_count = 0; h->prof_ev_made = false;
    return h;
}

commvq_status commvq_create_planner(const commvq_config *config, commvq_handle **out)
{
    if (!out) return COMMVQ_ERR_NULL;
    commvq_status st = commvq_validate_config(config);
    if (st != COMMVQ_OK) return st;
    commvq_handle *h = new_handle(config, -1);
    if (!h) return COMMVQ_ERR_LAUNCH;
    *out = h;
    return COMMVQ_OK;
}

commvq_status commvq_create(const commvq_config *config, commvq_handle **out)
{
    if (!out) return COMMVQ_ERR_NULL;
    commvq_status st = commvq_validate_config(config);
    if (st != COMMVQ_OK) return st;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); return COMMVQ_ERR_NO_DEVICE; }
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, dev) != hipSuccess) { (void)hipGetLastError(); return COMMVQ_ERR_NO_DEVICE; }
    if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0) return COMMVQ_ERR_NO_DEVICE;  // the kernels are gfx950 code only
    commvq_handle *h = new_handle(config, dev);
    if (!h) return COMMVQ_ERR_LAUNCH;
    // exact phases in fp64, rounded once to fp32
    std::vector<float2> hi((size_t)h->n_hi * kJ), lo((size_t)kLo * kJ);
    for (int j = 0; j < kJ; ++j) {
        const double theta = std::pow(config->rope_base, -2.0 * j / kD);
        for (int a = 0; a < h->n_hi; ++a) {
            const double ang = theta * (double)((int64_t)a << kLoBits);
            hi[(size_t)a * kJ + j] = make_float2((float)std::cos(ang), (float)std::sin(ang));
        }
        for (int a = 0; a < kLo; ++a) {
            const double ang = theta * (double)a;
            lo[(size_t)a * kJ + j] = make_float2((float)std::cos(ang), (float)std::sin(ang));
        }
    }
    bool ok = hipMalloc(reinterpret_cast<void **>(&h->tbl_hi), hi.size() * sizeof(float2)) == hipSuccess &&
              hipMalloc(reinterpret_cast<void **>(&h->tbl_lo), lo.size() * sizeof(float2)) == hipSuccess &&
              hipMemcpy(h->tbl_hi, hi.data(), hi.size() * sizeof(float2), hipMemcpyHostToDevice) == hipSuccess &&
              hipMemcpy(h->tbl_lo, lo.data(), lo.size() * sizeof(float2), hipMemcpyHostToDevice) == hipSuccess;
    // this device's address of the static scratch array (every GPU holds its own copy at its own address)
    void *sp = nullptr;
    ok = ok && hipGetSymbolAddress(&sp, HIP_SYMBOL(scratch)) == hipSuccess && sp != nullptr;
    h->static_scratch = sp;
    if (!ok) {
        (void)hipGetLastError();
        if (h->tbl_hi) (void)hipFree(h->tbl_hi);
        if (h->tbl_lo) (void)hipFree(h->tbl_lo);
        delete h;
        return COMMVQ_ERR_LAUNCH;
    }
    *out = h;
    return COMMVQ_OK;
}

commvq_status commvq_destroy(commvq_handle *h)
{
    if (!h) return COMMVQ_ERR_NULL;
    if (h->prof_ev_made)
        for (int i = 0; i < kProfRing; ++i)
            for (int k = 0; k < 4; ++k) (void)hipEventDestroy(h->prof_ev[i][k]);
    if (h->tbl_hi) (void)hipFree(h->tbl_hi);
    if (h->tbl_lo) (void)hipFree(h->tbl_lo);
    delete h;
    return COMMVQ_OK;
}

commvq_status commvq_plan_query(const commvq_handle *h, int32_t batch, int64_t total_tokens, int32_t max_seqlen,
                                commvq_plan *plan)
{
    if (!h || !plan) return COMMVQ_ERR_NULL;
    // explicit key positions are not known here: the distance check belongs to the calls that see them
    const commvq_status st = check_shape(h, batch, total_tokens, max_seqlen, true);
    if (st != COMMVQ_OK) return st;
    Plan p;
    make_plan(h, batch, total_tokens, max_seqlen, use_sliced(h, false), &p);
    *plan = p;
    return COMMVQ_OK;
}

commvq_status commvq_workspace_bytes(const commvq_handle *h, int32_t batch, int64_t total_tokens, int32_t max_seqlen,
                                     size_t *bytes)
{
    if (!bytes) return COMMVQ_ERR_NULL;
    commvq_plan plan;
    commvq_status st = commvq_plan_query(h, batch, total_tokens, max_seqlen, &plan);
    if (st != COMMVQ_OK) return st;
    Workspace w;
    carve(h, batch, total_tokens, max_seqlen, nullptr, &w);
    *bytes = w.bytes;
    return COMMVQ_OK;
}

commvq_status commvq_packed_key_codebook_bytes(const commvq_handle *h, size_t *bytes)
{
    if (!h || !bytes) return COMMVQ_ERR_NULL;
    if (h->cfg.codebook_dtype != COMMVQ_BF16) return COMMVQ_ERR_CONFIG;
    *bytes = packed_key_bytes(h->cfg);
    return COMMVQ_OK;
}

commvq_status commvq_pack_key_codebooks(commvq_handle *h, const void *key_cb, void *packed, void *stream)
{
    if (!h || !key_cb || !packed) return COMMVQ_ERR_NULL;
    if (h->cfg.codebook_dtype != COMMVQ_BF16) return COMMVQ_ERR_CONFIG;
    if ((reinterpret_cast<uintptr_t>(key_cb) | reinterpret_cast<uintptr_t>(packed)) & 15u) return COMMVQ_ERR_SHAPE;
    if (h->device < 0) return COMMVQ_ERR_NO_DEVICE;
    if (launch_prep(h->cfg, key_cb, static_cast<uint4 *>(packed), static_cast<hipStream_t>(stream)) != hipSuccess)
        return COMMVQ_ERR_LAUNCH;
    for (auto &e : h->packed_keys)
        if (e.first == key_cb) {
            e.second = static_cast<const uint4 *>(packed);
            return COMMVQ_OK;
        }
    try {
        h->packed_keys.emplace_back(key_cb, static_cast<const uint4 *>(packed));
    } catch (...) {
        return COMMVQ_ERR_LAUNCH;
    }
    return COMMVQ_OK;
}

commvq_status commvq_packed_value_codebook_bytes(const commvq_handle *h, size_t *bytes)
{
    if (!h || !bytes) return COMMVQ_ERR_NULL;
    if (h->cfg.codebook_dtype != COMMVQ_BF16) return COMMVQ_ERR_CONFIG;
    *bytes = (size_t)h->cfg.n_kv_heads * val_books(h->cfg) * kK * kD * 2;
    return COMMVQ_OK;
}

commvq_status commvq_pack_value_codebooks(commvq_handle *h, const void *val_cb, void *packed, void *stream)
{
    if (!h || !val_cb || !packed) return COMMVQ_ERR_NULL;
    if (h->cfg.codebook_dtype != COMMVQ_BF16) return COMMVQ_ERR_CONFIG;
    if ((reinterpret_cast<uintptr_t>(val_cb) | reinterpret_cast<uintptr_t>(packed)) & 15u) return COMMVQ_ERR_SHAPE;
    if (h->device < 0) return COMMVQ_ERR_NO_DEVICE;
    if (!bin_values(h->cfg)) return COMMVQ_OK;  // k_values reads the codebook as it is
    if (launch_prep_values(h->cfg, val_cb, static_cast<uint4 *>(packed), static_cast<hipStream_t>(stream)) != hipSuccess)
        return COMMVQ_ERR_LAUNCH;
    for (auto &e : h->packed_vals)
        if (e.first == val_cb) {
            e.second = static_cast<const uint4 *>(packed);
            return COMMVQ_OK;
        }
    try {
        h->packed_vals.emplace_back(val_cb, static_cast<const uint4 *>(packed));
    } catch (...) {
        return COMMVQ_ERR_LAUNCH;
    }
    return COMMVQ_OK;
}

commvq_status commvq_forget_packed_value_codebooks(commvq_handle *h, const void *val_cb)
{
    if (!h) return COMMVQ_ERR_NULL;
    for (size_t i = 0; i < h->packed_vals.size(); ++i)
        if (!val_cb || h->packed_vals[i].first == val_cb) {
            h->packed_vals.erase(h->packed_vals.begin() + (long)i);
            --i;
        }
    return COMMVQ_OK;
}

commvq_status commvq_forget_packed_key_codebooks(commvq_handle *h, const void *key_cb)
{
    if (!h) return COMMVQ_ERR_NULL;
    for (size_t i = 0; i < h->packed_keys.size(); ++i)
        if (!key_cb || h->packed_keys[i].first == key_cb) {
            h->packed_keys.erase(h->packed_keys.begin() + (long)i);
            --i;
        }
    return COMMVQ_OK;
}

commvq_status commvq_stage_scores(commvq_handle *h, const void *q, const uint8_t *key_codes, const void *key_cb,
                                  const commvq_positions *pos, void *workspace, size_t workspace_bytes,
                                  float *scores_out, void *stream)
{
    if (!h || !q || !key_codes || !key_cb) return COMMVQ_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(key_codes) & 15u) return COMMVQ_ERR_SHAPE;
    Plan plan;
    Workspace w;
    commvq_status st = prep(h, pos, workspace, workspace_bytes, &plan, &w);
    if (st != COMMVQ_OK) return st;
    hipStream_t s = static_cast<hipStream_t>(stream);
    st = run_scores(h, q, key_codes, key_cb, pos, plan, w, s);
    if (st != COMMVQ_OK) return st;
    if (scores_out &&
        hipMemcpyAsync(scores_out, w.scores, (size_t)pos->total_tokens * h->cfg.n_q_heads * sizeof(float),
                       hipMemcpyDeviceToDevice, s) != hipSuccess)
        return COMMVQ_ERR_LAUNCH;
    return COMMVQ_OK;
}

commvq_status commvq_stage_bins(commvq_handle *h, const uint8_t *val_codes, const commvq_positions *pos,
                                void *workspace, size_t workspace_bytes, void *stream)
{
    if (!h || !val_codes) return COMMVQ_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(val_codes) & 15u) return COMMVQ_ERR_SHAPE;
    Plan plan;
    Workspace w;
    commvq_status st = prep(h, pos, workspace, workspace_bytes, &plan, &w);
    if (st != COMMVQ_OK) return st;
    if (fused_values(h->cfg)) return run_values(h, val_codes, nullptr, pos, plan, w, 1, static_cast<hipStream_t>(stream));
    return run_bins(h, val_codes, pos, plan, w, static_cast<hipStream_t>(stream));
}

commvq_status commvq_stage_output(commvq_handle *h, const void *val_cb, const commvq_positions *pos, float *out,
                                  void *workspace, size_t workspace_bytes, void *stream)
{
    if (!h || !val_cb || !out) return COMMVQ_ERR_NULL;
    Plan plan;
    Workspace w;
    commvq_status st = prep(h, pos, workspace, workspace_bytes, &plan, &w);
    if (st != COMMVQ_OK) return st;
    if (fused_values(h->cfg)) {
        st = run_values(h, nullptr, val_cb, pos, plan, w, 2, static_cast<hipStream_t>(stream));
        return st == COMMVQ_OK ? run_values_final(h, pos, plan, w, out, static_cast<hipStream_t>(stream)) : st;
    }
    return run_output(h, val_cb, pos, plan, w, out, static_cast<hipStream_t>(stream));
}

commvq_status commvq_decode_attn(commvq_handle *h, const void *q, const uint8_t *key_codes, const uint8_t *val_codes,
                                 const void *key_cb, const void *val_cb, const commvq_positions *pos, float *out,
                                 void *workspace, size_t workspace_bytes, void *stream)
{
    if (!h || !q || !key_codes || !val_codes || !key_cb || !val_cb || !out) return COMMVQ_ERR_NULL;
    if ((reinterpret_cast<uintptr_t>(key_codes) | reinterpret_cast<uintptr_t>(val_codes)) & 15u) return COMMVQ_ERR_SHAPE;
    Plan plan;
    Workspace w;
    commvq_status st = prep(h, pos, workspace, workspace_bytes, &plan, &w);
    if (st != COMMVQ_OK) return st;
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipEvent_t *ev = nullptr;
    if (h->prof_every > 0 && h->prof_calls++ % h->prof_every == 0) {
        if (!h->prof_ev_made) {
            for (int i = 0; i < kProfRing; ++i)
                for (int k = 0; k < 4; ++k)
                    if (hipEventCreate(&h->prof_ev[i][k]) != hipSuccess) return COMMVQ_ERR_LAUNCH;
            h->prof_ev_made = true;
        }
        ev = h->prof_ev[h->prof_head];
        if (hipEventRecord(ev[0], s) != hipSuccess) return COMMVQ_ERR_LAUNCH;
    }
    st = run_scores(h, q, key_codes, key_cb, pos, plan, w, s);
    if (st != COMMVQ_OK) return st;
    if (ev && hipEventRecord(ev[1], s) != hipSuccess) return COMMVQ_ERR_LAUNCH;
    const bool fused = fused_values(h->cfg);
    st = fused ? run_values(h, val_codes, val_cb, pos, plan, w, 0, s) : run_bins(h, val_codes, pos, plan, w, s);
    if (st != COMMVQ_OK) return st;
    if (ev && hipEventRecord(ev[2], s) != hipSuccess) return COMMVQ_ERR_LAUNCH;
    st = fused ? run_values_final(h, pos, plan, w, out, s) : run_output(h, val_cb, pos, plan, w, out, s);
    if (st != COMMVQ_OK) return st;
    if (ev) {
        if (hipEventRecord(ev[3], s) != hipSuccess) return COMMVQ_ERR_LAUNCH;
        h->prof_head = (h->prof_head + 1) % kProfRing;
        if (h->prof_count < kProfRing) ++h->prof_count;
    }
    return COMMVQ_OK;
}

commvq_status commvq_decode_attn_static(commvq_handle *h, const void *q, const uint8_t *key_codes, const uint8_t *val_codes,
                                        const void *key_cb, const void *val_cb, const commvq_positions *pos, float *out,
                                        void *stream)
{
    if (!h || !q || !key_codes || !val_codes || !key_cb || !val_cb || !out) return COMMVQ_ERR_NULL;
    if ((reinterpret_cast<uintptr_t>(key_codes) | reinterpret_cast<uintptr_t>(val_codes)) & 15u) return COMMVQ_ERR_SHAPE;
    Plan plan;
    Workspace w;
    // the handle's copy of the scratch array is the workspace; a batch shape that needs more than the array holds
    // comes back as COMMVQ_ERR_WORKSPACE from the same check that vets a caller's workspace
    commvq_status st = prep(h, pos, h->device < 0 ? reinterpret_cast<void *>(256) : h->static_scratch, kStaticScratchBytes, &plan, &w);
    if (st != COMMVQ_OK) return st;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev != h->device) return COMMVQ_ERR_NO_DEVICE;  // the array of another GPU
    hipStream_t s = static_cast<hipStream_t>(stream);
    st = run_scores(h, q, key_codes, key_cb, pos, plan, w, s);
    if (st != COMMVQ_OK) return st;
    const bool fused = fused_values(h->cfg);
    st = fused ? run_values(h, val_codes, val_cb, pos, plan, w, 0, s) : run_bins(h, val_codes, pos, plan, w, s);
    if (st != COMMVQ_OK) return st;
    return fused ? run_values_final(h, pos, plan, w, out, s) : run_output(h, val_cb, pos, plan, w, out, s);
}

commvq_status commvq_static_scratch_bytes(size_t *bytes)
{
    if (!bytes) return COMMVQ_ERR_NULL;
    *bytes = kStaticScratchBytes;
    return COMMVQ_OK;
}

commvq_status commvq_profile_enable(commvq_handle *h, int32_t every)
{
    if (!h) return COMMVQ_ERR_NULL;
    h->prof_every = every > 0 ? every : 0;
    h->prof_calls = 0;
    h->prof_head = h->prof_count = 0;
    return COMMVQ_OK;
}

commvq_status commvq_profile_read(commvq_handle *h, float *mean_ms, int32_t *n_calls)
{
    if (!h || !mean_ms || !n_calls) return COMMVQ_ERR_NULL;
    double acc[3] = {0, 0, 0};
    const int n = h->prof_count;
    for (int k = 0; k < n; ++k) {
        const int i = (h->prof_head - 1 - k + 2 * kProfRing) % kProfRing;
        if (hipEventSynchronize(h->prof_ev[i][3]) != hipSuccess) return COMMVQ_ERR_LAUNCH;
        for (int st = 0; st < 3; ++st) {
            float ms = 0.f;
            if (hipEventElapsedTime(&ms, h->prof_ev[i][st], h->prof_ev[i][st + 1]) != hipSuccess) return COMMVQ_ERR_LAUNCH;
            acc[st] += ms;
        }
    }
    for (int st = 0; st < 3; ++st) mean_ms[st] = n ? (float)(acc[st] / n) : 0.f;
    *n_calls = n;
    h->prof_head = h->prof_count = 0;
    return COMMVQ_OK;
}

}  // extern "C"
