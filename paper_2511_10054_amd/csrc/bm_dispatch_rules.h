// Rules on sizes that choose between kernels: which batches stream and which are tiled, which decode layers take the two-wave
// form of the LDS-staged streaming kernel, projection by projection, where the stand-alone substitution takes one workgroup, and how far apart the
// grouping kernels' sets lie.  Plain C++ without HIP, so that a host test can look at the choices.
#pragma once
#include "../../include/buddymoe.h"

namespace bm {

// Layers of many small experts at up to 32 tokens: the LDS-staged streaming kernel with two-wave workgroups
// (32 weight rows), because 64-row blocks leave compute units without one.  ms with four waves | two waves,
// Qwen3-shaped layer (E = 128, d = 2048, F = 768) at 2 / 8 / 16 / 32 / 64 tokens: .051 .060 .076 .086 .102 | .047
// .059 .071 .082 .106; Mixtral-shaped (F = 14336, 224 blocks of 64 rows per expert) at 8 / 32 tokens .234 .319 |
// .259 .324.  The line between the two lies at matrices of 16 MB and F = 2048.
// With more than some 500 blocks of 64 rows the two are within 5 % of each other either way, by how the live groups
// (which the host does not know) divide among the units; the mean over 300 shapes is 1.00.
inline bool narrow_shape(const bm_layer_desc *d) {
    return d->dtype == BM_BF16 && d->T <= 32 && d->d % 128 == 0 && d->F % 128 == 0 && d->F <= 2048 &&
           (long long)d->d * d->F <= (1ll << 23);
}

// The most groups (expert matrices) that a batch reads
inline long long decode_groups(const bm_layer_desc *d) {
    const long long rows = (long long)d->T * d->K;
    return (rows < d->E ? rows : d->E) + (d->n_shared > 0 ? d->n_shared : 0);
}

// A projection [N][Kd] of few groups whose reduction the quarter-split kernel takes (multiples of 1024, up to 32 rows): its
// workgroups of 16 rows, four waves along the reduction, are twice as many with twice the waves.  Two-wave | quarter-split
// layers, us, cold weights: 8 experts, K = 2, d = 1024, F = 1024 at 1 / 2 tokens (64 / 128 two-wave workgroups a
// projection) 21.1 21.6 | 18.9 19.6; d = 2048 at 1 token (128) 22.6 | 21.2; one expert a token, d = 3072 (96) 28.9 |
// 26.0, d = 4096 (128) 25.8 | 24.3; d = 1024, K = 5 (160) 23.5 | 24.7, K = 6 (192) 24.4 | 25.7.
inline bool quarter_split_projection(const bm_layer_desc *d, int N, int Kd) {
    return Kd % 1024 == 0 && (long long)d->T * d->K <= 32 && decode_groups(d) * (N / 32) <= 128;
}

// F = 2048 past 32 rows: the down projection is long enough to be split into two slices of the reduction, and from 512
// gate/up blocks of 64 rows on no unit is without one.  Two waves for both | four waves for both (split) | two-wave gate/up
// and split down, us: d = 4096, 16 experts, K = 4 at 9 / 16 / 32 tokens 157 165 161 | 144 154 157 | 152 159 156; 32
// experts at 32 tokens 299 | 282 | 292; d = 3072, 4 experts, K = 2 at 24 tokens 45 | 51 | 46; 8 experts 69 | 69 | 69.
// Only where the four-wave form takes the gate/up reduction (multiples of 256): else gate/up has nowhere faster to go, and
// the split alone is within 4 % either way.
inline bool long_narrow(const bm_layer_desc *d) { return d->F >= 2048 && d->d % 256 == 0 && (long long)d->T * d->K > 32; }

inline bool narrow_gateup(const bm_layer_desc *d) {
    return narrow_shape(d) && !quarter_split_projection(d, d->F, d->d) &&
           !(long_narrow(d) && decode_groups(d) * (d->F / 64) >= 512);
}
// the reduction of the down projection stays whole (one fp32 output); compact: whatever needs the least scratch
inline bool narrow_down_whole(const bm_layer_desc *d, bool compact) {
    return narrow_shape(d) && (compact || !long_narrow(d));
}
inline bool narrow_down(const bm_layer_desc *d, bool compact) {
    return narrow_down_whole(d, compact) && !quarter_split_projection(d, d->d, d->F);
}

// Shapes both projections of which fit the persistent k-step-64 kernel: reduction widths that are multiples
// of 64 and at least 256, operands within 32-bit byte offsets.
inline bool k64_shape(const bm_layer_desc *d) {
    const unsigned long long lim = 1ull << 32;
    const int ns = d->n_shared > 0 ? d->n_shared : 0;
    const unsigned long long rows = (unsigned long long)d->T * (d->K + ns) + 256ull * (d->E + ns);
    return d->dtype == BM_BF16 && d->d % 64 == 0 && d->F % 64 == 0 && d->d >= 256 && d->F >= 256 &&
           (unsigned long long)d->T * d->d * 2 < lim && rows * d->F * 2 < lim && (unsigned long long)d->F * d->d * 2 < lim;
}

constexpr int SKINNY_MAX_ROWS = 256;   // total rows up to which the weight-streaming path is always used,
constexpr int SKINNY_AVG_ROWS = 16;    // ... and rows per group (averaged over all experts) likewise
constexpr int SKINNY_UNFIT_ROWS = 16;  // total rows when the widths do not fit its fast kernels but do fit the persistent tiled kernel

// Widths that are multiples of 128 but not of 256 take the two-wave streaming kernel (narrow_shape) instead of the
// tiled path up to 16 tokens
// (DeepSeek-shaped layer, F = 1408, at 3 / 8 / 16 / 32 tokens: tiled .061 .077 .080 .087, two-wave streaming .053
// .062 .070 .089), as long as its fp32 down-projection output is small (the tiled path's is bf16).  A call whose
// workspace has no room for that output keeps the tiled path (plan_layout): one that is sized for the largest batch
// of a serving loop, of 17 to 25 tokens for instance, takes every smaller batch.
constexpr int NARROW_UNFIT_T = 16;
constexpr long long NARROW_UNFIT_BYTES = 16ll << 20;

// Few rows per group: every expert group is decode-sized and the projections are bound by reading the
// weights once.  Up to 256 rows in all, or up to 16 rows per expert on average (Qwen3-shaped layer, 128
// experts, 64 / 128 / 256 tokens: 0.11 / 0.13 / 0.16 ms against 0.14 / 0.15 / 0.16 ms on the tiled path), when
// both widths fit the fast streaming kernels (multiples of 256).  Widths that do not (DeepSeek-shaped layer,
// F = 1408, whose shared experts take every token as well) leave the streaming path to its slower
// fallbacks: there the persistent tiled kernel is faster from 4 tokens on (4 / 8 / 32 tokens: 0.064 / 0.071 /
// 0.089 against 0.068 / 0.082 / 0.101 ms), so the streaming path keeps only batches of at most 16 rows, unless
// the two-wave kernel takes the shape (narrow_shape).
// Streaming | tiled, us: Mixtral-shaped layer 64 / 96 / 112 / 128 tokens, public weights 338 364 373 411 | 341 354 355 356,
// packed 311 340 346 364 | 345 354 351 357; Qwen3-shaped 128 / 192 / 224 / 256 tokens 112 134 145 153 | 132 135 139 140.
// The batches at the upper end would be faster tiled, but that path holds the down projection's output in bf16 until
// the aggregation, the streaming one in fp32 (error against 64 bits 0.0029 | 0.0023), so the lines stay where they are.
inline bool use_skinny(const bm_layer_desc *d, bool compact) {
    if (d->dtype != BM_BF16) return false;
    const int ns = d->n_shared > 0 ? d->n_shared : 0;
    const long long rows = (long long)d->T * (d->K + ns);
    const bool fit = d->d % 256 == 0 && d->F % 256 == 0;
    if (!fit && k64_shape(d))
        return rows <= SKINNY_UNFIT_ROWS || (!compact && narrow_shape(d) && d->T <= NARROW_UNFIT_T && rows * (2ll * d->F + 4ll * d->d) <= NARROW_UNFIT_BYTES);
    if (rows <= SKINNY_MAX_ROWS) return true;
    return fit && rows <= (long long)SKINNY_AVG_ROWS * (d->E + ns);
}

// Most live groups whose three matrices the 256 MB memory-side cache holds until the layer's next call.  The tiled kernels
// load weights that are read once non-temporally where a batch has more live groups than that (a count that the grouping leaves on
// the device: most experts of a layer may be absent).  us, plain | non-temporal, warm, bf16: 16 of 64 experts resident, d = F = 1024, 101 MB
// of 403, 600 / 1500 / 3000 tokens 54 69 96 | 57 72 102; 24 of 96, d = 1024, F = 512, 75 MB of 302, 1000 / 3000 tokens 57 73 |
// 59 75; 48 of 48, d = F = 1024, 302 MB, level; Qwen3-shaped, 604 MB, 512 tokens gate/up 85 | 79.
constexpr long long MEMORY_SIDE_CACHE = 256ll << 20;
inline int cached_groups(const bm_layer_desc *d) {
    return (int)(MEMORY_SIDE_CACHE / ((d->dtype == BM_BF16 ? 6ll : 12ll) * d->d * d->F));
}

// Tokens of a tile of the stand-alone substitution kernel, and the most tokens that a single workgroup takes.  It stores
// the counters itself and needs no launch in front of it that zeroes them (1.8 us), but takes the tiles one after the
// other.  One workgroup | one per tile, us: 8 of 128 experts, no ties between a token's slots, 65 / 128 / 192 tokens 5.9
// 6.6 8.3 | 6.7 6.8 6.9; U_t, 65 / 96 / 128 / 192 tokens 8.3 8.4 10.2 13.6 | 8.7 8.3 8.6 8.7; more than eight slots,
// which a lane walks (16 of 256 experts), 64 / 65 / 96 tokens 22.6 32.4 38.0 | - 24.1 23.7.
constexpr int REMAP_TOK = 64;
inline int remap_one_workgroup_tokens(int K, uint32_t flags) {
    if (!(flags & (BM_REMAP_UNIQUE | BM_GATE_ANY | BM_PSI_TOKEN))) return 2 * REMAP_TOK;
    return K <= 8 && !(flags & BM_PSI_TOKEN) ? 96 : REMAP_TOK;
}

// Co-activation counts in chunks of 512 tokens instead of 1024: better while the additions to the totals are few or the tokens'
// slots many.  Time of 512 over 1024, calls of a captured graph (from Python a call takes 7.3 us to issue, more than most of these
// run), at 1000 / 2048 / 4096 / 8192 / 16384 tokens: up to 8 slots of 8 or 16 experts .90 .89 .90 .93 1.00 (32768: 1.11); 4 slots of
// 64 experts .91 .97 1.07 1.23 1.38, of 256 .95 .98 1.07 1.20 1.05; 8 slots of 16 experts .71 .71 .71 .74 .78, of 64 .74 .78 .85
// .99 1.16, of 128 .75 .80 .88 1.02 1.08, of 256 .81 .87 1.00 1.15 .94 (8192 tokens 12.1 us in chunks of 1024).
inline bool coact_short_chunks(int T, int K, int E) {
    return T <= 2048 || (K >= 8 ? (long long)T * E <= 1 << 19 : E <= 16 && T <= 16384);
}

// Words between the assignment sets of consecutive experts in LDS, for A assignments (bit a % 64 of word a / 64).  Long sets
// lie an odd number of words apart: at 16 or 32 words the same word of every expert's set is in one bank (grouping of
// 1024 / 2048 assignments of 16 experts 6.0 13.8 us, an odd number 4.6 6.1; layers of 8 experts, 2048 assignments 45.4 -> 41.0).
constexpr int set_stride(int A) {
    const int words = (A + 63) >> 6;
    return words >= 8 ? words | 1 : words;
}

}  // namespace bm
