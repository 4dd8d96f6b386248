// Front end of the layer: router logits, softmax / top-k gates, buddy
// substitution (Section 4, Algorithm 1) and the stable grouping of the
// surviving assignments by expert.
//
// Tokens are processed in tiles of TILE_T = 32 (16 for fp32 and for bf16 batches
// of up to 8160 tokens, see front_tile_tokens).  One workgroup owns one tile:
// its waves split the hidden dimension for the router product (MFMA,
// for bf16 and fp32; few tokens and many experts: in a launch of its own), the
// partial logits meet in LDS, then each wave ranks
// whole tokens (one expert per lane), Algorithm 1 runs on eight lanes per token
// (remap_tile; more than eight slots, or priorities: a lane walks the slots),
// and the tile's per-expert histogram goes to global memory.  One kernel, or a
// one-workgroup scan and a scatter kernel for large histograms, turns the
// histograms into group offsets, the row-tile table of the grouped GEMMs and the
// position of every assignment (rank inside the tile from its expert's
// assignment set, so the order is the stable one and no atomics decide a
// position).  Small batches get offsets and placement from one workgroup instead
// (group_small_kernel), or from the front kernel itself (FUSED, or the tail of a
// single tile).
#include "bm_dispatch_rules.h"
#include "bm_kernels.h"

#include <type_traits>

namespace bm {

// ---------------------------------------------------------------------------
// Sets of experts (the residency mask, a token's U_t) in W words of 64; W = ceil(E / 64) is known at compile time,
// because picking one of four words costs most of a test.
// ---------------------------------------------------------------------------
template <int W>
__device__ __forceinline__ bool test_bit(const uint64_t (&m)[W], int b) {
    uint64_t wv = m[0];
#pragma unroll
    for (int i = 1; i < W; ++i) {
        const uint64_t mi = m[i];        // read whatever the condition: the conditional read of one of four becomes an
        wv = (b >> 6) == i ? mi : wv;    // indexed one, which puts the array into scratch memory
    }
    return (wv >> (b & 63)) & 1ull;
}

// Gates in front of the substitution (Section 3.1: TAE, Eq. 1, and probability margin;
// Section 5.1: replacement budget).  From the token's K gate weights renormalised to sum 1:
// the token may be given substitutes unless (BM_GATE_TAE and TAE <= tau) or (BM_GATE_MARGIN and
// largest - second largest >= gamma); returns how many slots may be replaced (0 = none).
// (eight weights at a time, so that their reads, divisions and logarithms overlap; the sums stay in slot order)
__device__ __forceinline__ int replacement_budget(int K, uint32_t flags, float tau, float gamma, int rho,
                                                  const float *w) {
    int budget = (flags & BM_REPLACE_BUDGET) ? rho : 0x7fffffff;
    if (flags & (BM_GATE_TAE | BM_GATE_MARGIN)) {
        float sum = 0.0f;
        for (int k0 = 0; k0 < K; k0 += 8) {
            float v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = w[min(k0 + i, K - 1)];
#pragma unroll
            for (int i = 0; i < 8; ++i) sum = k0 + i < K ? sum + v[i] : sum;
        }
        float h = 0.0f, p1 = 0.0f, p2 = 0.0f;
        for (int k0 = 0; k0 < K; k0 += 8) {
            float pk[8], t[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) pk[i] = w[min(k0 + i, K - 1)] / sum;
#pragma unroll
            for (int i = 0; i < 8; ++i) t[i] = pk[i] > 0.0f ? pk[i] * logf(pk[i]) : 0.0f;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                if (k0 + i >= K) break;
                h -= t[i];
                const float lo = fminf(p1, pk[i]);
                p1 = fmaxf(p1, pk[i]);
                p2 = fmaxf(p2, lo);
            }
        }
        const float tae = K > 1 ? h / logf((float)K) : 0.0f;
        if ((flags & BM_GATE_TAE) && tae <= tau) budget = 0;
        if ((flags & BM_GATE_MARGIN) && (p1 - p2) >= gamma) budget = 0;
    }
    return budget;
}

// Distribution gate (Section 3.1, Eq. 2): delta = n_cpu / n_req >= beta, decided without rounding
// (both products are exact in fp64 for counts up to BM_MAX_E and an fp32 threshold).
__device__ __forceinline__ bool dist_bypass(int n_req, int n_cpu, float beta) {
    return n_req > 0 && (double)n_cpu >= (double)beta * (double)n_req;
}

// Token-aware buddy priority (Section 3.1, Eq. 3 with kappa = 0): how the normalised router logit of
// expert b (its softmax probability over all experts) is obtained for token t of the tile at hand.
struct PsiSource {
    const float *q;        // [E][R] q[j|i] of every table entry; null: priority = table order
    float eta;
    int stride;            // between the tokens of logits or probs
    const float *logits;   // logit rows (bias included), with zmax and inv_den per token; or null
    const float *zmax, *inv_den;
    const float *probs;    // probability rows; used when logits is null
    __device__ __forceinline__ float zhat(int t, int b) const {
        return logits != nullptr ? __expf(logits[t * stride + b] - zmax[t]) * inv_den[t] : probs[(size_t)t * stride + b];
    }
};

// Entries of a buddy row that may stand in for its expert: bit r set if entry r < H is in [0, E) and resident.
// (8 entries at a time: the reads of a batch go out together)
template <int W>
__device__ __forceinline__ uint32_t acceptable_entries(const int32_t *row, int H, int E, const uint64_t (&resident)[W]) {
    uint32_t m = 0;
    for (int r0 = 0; r0 < H; r0 += 8) {
        int b[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) b[i] = row[min(r0 + i, H - 1)];       // (no branches between the reads)
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (r0 + i < H && (unsigned)b[i] < (unsigned)E && test_bit<W>(resident, b[i])) m |= 1u << (r0 + i);
    }
    return m;
}

// v of the lanes ^ 0 .. ^ 7 inside each group of eight (quad permutes, and a mirror of eight for the upper four)
__device__ __forceinline__ void lanes_of_eight(int v, int (&out)[8]) {
#define BM_DPP_MOV(v_, ctrl_) __builtin_amdgcn_update_dpp(0, v_, ctrl_, 0xF, 0xF, true)
    out[0] = v;
    out[1] = BM_DPP_MOV(v, 0xB1);
    out[2] = BM_DPP_MOV(v, 0x4E);
    out[3] = BM_DPP_MOV(v, 0x1B);
    out[7] = BM_DPP_MOV(v, 0x141);
    out[6] = BM_DPP_MOV(out[7], 0xB1);
    out[5] = BM_DPP_MOV(out[7], 0x4E);
    out[4] = BM_DPP_MOV(out[7], 0x1B);
#undef BM_DPP_MOV
}

// replacement_budget() for a token held by eight lanes, lane k with the gate weight of slot k (KC = 1: by one lane): the same
// operations in the same order, the divisions and logarithms of the slots side by side.
template <int KC>
__device__ __forceinline__ int replacement_budget_of_eight(int K, int k, uint32_t flags, float tau, float gamma, int rho, float wk) {
    int budget = (flags & BM_REPLACE_BUDGET) ? rho : 0x7fffffff;
    if (flags & (BM_GATE_TAE | BM_GATE_MARGIN)) {
        const int first = KC == 1 ? lane_id() : lane_id() & 56;
        float h = 0.0f, p1 = 0.0f, p2 = 0.0f;
        auto evaluate = [&](auto slots) {                // the first so many lanes, K of them with a slot
            constexpr int N = decltype(slots)::value;
            float v[N], sum = 0.0f;
#pragma unroll
            for (int j = 0; j < N; ++j) v[j] = __shfl(wk, first + j, WAVE);
#pragma unroll
            for (int j = 0; j < N; ++j) sum = j < K ? sum + v[j] : sum;
            const float mine = k < K ? wk / sum : 0.0f;
            const float term = mine > 0.0f ? mine * logf(mine) : 0.0f;
#pragma unroll
            for (int j = 0; j < N; ++j) {
                const float pj = __shfl(mine, first + j, WAVE), tj = __shfl(term, first + j, WAVE);
                if (j >= K) continue;
                h -= tj;
                const float lo = fminf(p1, pj);
                p1 = fmaxf(p1, pj);
                p2 = fmaxf(p2, lo);
            }
        };
        if (K <= 2) evaluate(std::integral_constant<int, KC == 1 ? 1 : 2>{});
        else evaluate(std::integral_constant<int, 8>{});
        const float tae = K > 1 ? h / logf((float)K) : 0.0f;
        if ((flags & BM_GATE_TAE) && tae <= tau) budget = 0;
        if ((flags & BM_GATE_MARGIN) && (p1 - p2) >= gamma) budget = 0;
    }
    return budget;
}

// Algorithm 1 for a tile of tokens; every thread of the workgroup calls it.  ids [ntok][K] sits in LDS, the router's
// choice in, the substituted ids (-1 dropped) out; `accept` holds acceptable_entries() of every expert; `used`
// is LDS scratch of ntok * W words (U_t: the tokens' original ids; read with BM_REMAP_UNIQUE only).
//   1. a thread per assignment finds the candidate: the first acceptable entry that is not one of the token's
//      original ids.  The assignment becomes expert | candidate << 8 | entry << 16 | PICK_* flags.
//   2. a lane per token walks its slots in order: budget, and - where an earlier slot has just been given the
//      candidate - the row's next acceptable entry.  What the walk reads is fetched eight slots at a time.
// One lane's walk is a chain of dependent instructions of a few cycles each, so as much as possible happens in step 1
// (8 tokens, 8 slots each, 128 experts: all of it in the walk 4.7 us).
//
// Without priorities the slots of a token are tied together by U_t and the budget only, and up to eight slots - eight
// lanes hold a token then - need no walk.  U_t: every lane sees the other slots' ids and candidates through DPP
// moves, and as long as two slots hold the same candidate, the lowest slot that shares one with an earlier slot
// moves on to its row's next entry (all slots before it are final then, so this is the order of the algorithm;
// mostly no or one turn).  The budget, from gates evaluated once per token, keeps the first so many substitutes in
// slot order.  Without U_t and gates any number of slots goes that way, a lane per assignment; so does a single slot per
// token, compiled for it (KC = 1; 1 of 64 experts behind the gates, 1024 / 16384 tokens: 5.5 8.2 us, in eight lanes 8.2 10.7).
// (bm_buddy_remap of 4096 tokens of 8 out of 128 experts with U_t: 9.0 us; 28 us with all of it in a lane's walk.)
constexpr int PICK_RESIDENT = 1 << 24, PICK_CANDIDATE = 1 << 25, PICK_VALID = 1 << 26;

template <int W, int KC = 0>
__device__ __forceinline__ void remap_tile(int ntok, int K_, int E, int R, uint32_t flags, float tau, float gamma, int rho,
                                           const uint64_t (&resident)[W], const uint32_t *accept, const int32_t *table,
                                           int32_t *ids, float *w, unsigned long long *used, int32_t *stats,
                                           const PsiSource &psi) {
    const int tid = threadIdx.x, K = KC != 0 ? KC : K_, n = ntok * K;
    const bool unique = (flags & BM_REMAP_UNIQUE) != 0 && K > 1;       // (a single slot's own id is not resident, so no candidate)
    const bool tied = unique || (flags & BM_GATE_ANY) != 0;
    if (psi.q == nullptr && (!tied || K <= 8)) {
        const int per = tied && KC != 1 ? 8 : K, total = ntok * per;   // lanes per token
        for (int i0 = 0; i0 < total; i0 += blockDim.x) {
            const int i = i0 + tid, t = i / per, k = i - t * per;
            const bool slot = i < total && k < K;
            const int e = slot ? ids[t * K + k] : -1;
            const bool valid = (unsigned)e < (unsigned)E, res = valid && test_bit<W>(resident, e);
            const int32_t *row = table + (size_t)(valid ? e : 0) * R;
            uint32_t m = valid && !res ? accept[e] : 0u;               // entries left to try; the candidate is the lowest
            int cand = m != 0u ? row[__builtin_ctz(m)] : -1;
            if (unique) {
                int held[8], other[8];                                 // from lane ^ 0 .. lane ^ 7
                lanes_of_eight(valid ? e : -1, held);
                auto skip_held = [&]() {                               // the token's original ids stay in U_t
                    while (m != 0u) {
                        bool in = false;
#pragma unroll
                        for (int j = 0; j < 8; ++j) in |= held[j] == cand;
                        if (!in) break;
                        m &= m - 1;
                        cand = m != 0u ? row[__builtin_ctz(m)] : -1;
                    }
                };
                skip_held();
                for (;;) {
                    lanes_of_eight(cand, other);
                    bool shared = false;
#pragma unroll
                    for (int j = 1; j < 8; ++j) shared |= ((k ^ j) < k) & (other[j] == cand);
                    const unsigned long long all = __ballot(shared && cand >= 0);
                    if (all == 0ull) break;
                    const unsigned mine = (unsigned)(all >> (tid & 56)) & 255u;
                    if (shared && cand >= 0 && (mine & ((1u << k) - 1u)) == 0u) {
                        m &= m - 1;
                        cand = m != 0u ? row[__builtin_ctz(m)] : -1;
                        skip_held();
                    }
                }
            }
            if (flags & BM_GATE_ANY) {
                const int budget = replacement_budget_of_eight<KC>(K, k, flags, tau, gamma, rho, w != nullptr && slot ? w[(size_t)t * K + k] : 0.0f);
                const unsigned taken = (unsigned)(__ballot(cand >= 0) >> (tid & 56)) & ((1u << k) - 1u);
                if (__popc(taken) >= budget) cand = -1;
            }
            const int out = res ? e : cand;
            if (slot) {
                ids[t * K + k] = out;
                if (w != nullptr && out < 0) w[(size_t)t * K + k] = 0.0f;
            }
            const int n_miss = __popcll(__ballot(valid && !res)), n_sub = __popcll(__ballot(valid && !res && cand >= 0));
            if ((tid & 63) == 0 && n_miss) {
                atomicAdd(&stats[0], n_miss);
                atomicAdd(&stats[1], n_sub);
                atomicAdd(&stats[2], n_miss - n_sub);
            }
        }
        __syncthreads();
        return;
    }
    if (unique) {
        for (int i = tid; i < ntok * W; i += blockDim.x) used[i] = 0ull;
        __syncthreads();
        for (int idx = tid; idx < n; idx += blockDim.x) {
            const int e = ids[idx];
            if ((unsigned)e < (unsigned)E) atomicOr(&used[(idx / K) * W + (e >> 6)], 1ull << (e & 63));
        }
        __syncthreads();
    }
    for (int idx = tid; idx < n; idx += blockDim.x) {
        const int e = ids[idx];
        int v = 0;
        if ((unsigned)e < (unsigned)E) {
            v = e | PICK_VALID;
            if (test_bit<W>(resident, e)) v |= PICK_RESIDENT;
            else if (psi.q == nullptr) {
                const unsigned long long *u = used + (idx / K) * W;
                for (uint32_t m = accept[e]; m != 0u; m &= m - 1) {
                    const int r = __builtin_ctz(m), b = table[(size_t)e * R + r];
                    if (unique && ((u[b >> 6] >> (b & 63)) & 1ull)) continue;
                    v |= PICK_CANDIDATE | b << 8 | r << 16;
                    break;
                }
            }
        }
        ids[idx] = v;
    }
    __syncthreads();
    if (tid < ntok) {
        int32_t *tok = ids + tid * K;
        float *tw = w != nullptr ? w + (size_t)tid * K : nullptr;
        const unsigned long long *u = used + tid * W;
        int n_miss = 0, n_sub = 0, budget = 0x7fffffff;
        if (flags & BM_GATE_ANY) budget = replacement_budget(K, flags, tau, gamma, rho, tw);      // before any drop
        uint64_t given[W] = {};                            // substitutes of the earlier slots
        for (int k0 = 0; k0 < K; k0 += 8) {
            int v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = tok[min(k0 + i, K - 1)];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                if (k0 + i >= K) break;
                const bool miss = (v[i] & (PICK_VALID | PICK_RESIDENT)) == PICK_VALID;
                const int32_t *row = table + (size_t)(v[i] & 255) * R;
                int cand = (v[i] >> 8) & 255;
                bool ok = miss && (v[i] & PICK_CANDIDATE) != 0 && budget > 0;      // else used up or gated: no search
                if (psi.q != nullptr) {
                    // the acceptable entry of largest q * (1 + eta * zhat); equal scores keep the earlier entry
                    if (miss && budget > 0) {
                        const float *qrow = psi.q + (size_t)(v[i] & 255) * R;
                        float best = 0.0f;
                        for (uint32_t m = accept[v[i] & 255]; m != 0u; m &= m - 1) {
                            const int r = __builtin_ctz(m), b = row[r];
                            if (unique && (((u[b >> 6] >> (b & 63)) & 1ull) || test_bit<W>(given, b))) continue;
                            const float score = qrow[r] * (1.0f + psi.eta * psi.zhat(tid, b));
                            if (!ok || score > best) { cand = b; best = score; ok = true; }
                        }
                    }
                } else if (unique && __any(ok && test_bit<W>(given, cand))) {      // rare: one branch for the wave
                    if (ok && test_bit<W>(given, cand)) {
                        ok = false;
                        for (uint32_t m = accept[v[i] & 255] & ~((2u << ((v[i] >> 16) & 31)) - 1u); m != 0u; m &= m - 1) {
                            const int b = row[__builtin_ctz(m)];
                            if (((u[b >> 6] >> (b & 63)) & 1ull) || test_bit<W>(given, b)) continue;
                            cand = b;
                            ok = true;
                            break;
                        }
                    }
                }
                if (unique) {                              // without U_t nobody asks
#pragma unroll
                    for (int c = 0; c < W; ++c) given[c] |= ok && (W == 1 || (cand >> 6) == c) ? 1ull << (cand & 63) : 0ull;
                }
                n_miss += miss ? 1 : 0;
                n_sub += ok ? 1 : 0;
                budget -= ok ? 1 : 0;
                const int out = ok ? cand : (v[i] & PICK_RESIDENT) ? (v[i] & 255) : -1;
                tok[k0 + i] = out;
                if (tw != nullptr && out < 0) tw[k0 + i] = 0.0f;
            }
        }
        if (n_miss) atomicAdd(&stats[0], n_miss);
        if (n_sub) atomicAdd(&stats[1], n_sub);
        if (n_miss - n_sub) atomicAdd(&stats[2], n_miss - n_sub);
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// Shared LDS block of the front kernels.
// ---------------------------------------------------------------------------
struct FrontLds {
    alignas(16) int32_t ids[TILE_T * BM_MAX_K];
    float w[TILE_T * BM_MAX_K];
    unsigned long long used[TILE_T * 4];
    int32_t counts[BM_MAX_E];
    int32_t lut[BM_MAX_E];
    int32_t stats[4];
    int32_t dist[4];         // distribution gate: requested, requested and offloaded, bypassed
    uint64_t bitmap[4];
    unsigned long long req[4];
    float zmax[TILE_T], inv_den[TILE_T];   // per token: largest logit, 1 / sum of exp over all experts
};

// Ranks the tile's tokens from the logits in LDS and finishes the tile.
// logits: [TILE_T][stride] fp32, bias already added.  The logits region is
// reused for the buddy table once ranking is done (cap = its size in ints).
template <int EC>   // EC = ceil(E / 64) experts per lane (compile-time bound)
__device__ void tile_epilogue(const FrontParams &p, float *logits, int stride, int cap_ints,
                              FrontLds &s, int tile) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = blockDim.x >> 6;
    const int t0 = tile * p.tile_tokens;
    const int ntok = min(p.tile_tokens, p.T - t0);
    const int E = p.E, K = p.K;
    const int ec = (E + 63) >> 6;

    // Lane l owns experts l, l+64, ...  Few experts - ranking by counting: the rank of an expert is the
    // number of experts that beat it (larger logit, or equal logit and lower index), found with E
    // broadcast reads of the logit row, no cross-lane traffic; experts of rank < K are the selection,
    // slot = rank.  Many experts - K rounds of a wave-wide maximum (see below).  Same order either way.
    for (int i = wave; i < ntok; i += nw) {
        const float *zr = logits + i * stride;
        float myv[EC];
        int rank[EC];
#pragma unroll
        for (int c = 0; c < EC; ++c) {
            const int e = lane + 64 * c;
            myv[c] = (e < E) ? zr[e] : -INFINITY;
            rank[c] = 0;
        }
        if (E <= 16) {
#pragma unroll 16
            for (int j = 0; j < E; ++j) {              // branch-free body, unrolled: the LDS reads go out in batches
                const float zj = zr[j];
#pragma unroll
                for (int c = 0; c < EC; ++c)
                    rank[c] += (int)(zj > myv[c]) | ((int)(zj == myv[c]) & (int)(j < lane + 64 * c));
            }
#pragma unroll
            for (int c = 0; c < EC; ++c) {
                const int e = lane + 64 * c;
                if (e < E && rank[c] < K) {
                    s.ids[i * K + rank[c]] = e;
                    s.w[i * K + rank[c]] = myv[c];        // the logit for now; replaced by the gate weight below
                }
            }
        } else {
            // Many experts: K rounds of "largest remaining" instead (counting costs E reads per lane).
            // A round takes the wave-wide maximum of the order-preserving integer image of the logits,
            // then the lowest expert index that holds it (ballots, lowest set lane of the lowest c);
            // that expert's owner takes it out of the race (0 is below the image of every float).
            uint32_t key[EC];
#pragma unroll
            for (int c = 0; c < EC; ++c) key[c] = (lane + 64 * c < E) ? float_to_ordered(myv[c]) : 0u;
            int win = 0;                                   // lane r: the winner of round r
            uint32_t won = 0u;
            for (int r = 0; r < K; ++r) {
                uint32_t mine = key[0];
#pragma unroll
                for (int c = 1; c < EC; ++c) mine = key[c] > mine ? key[c] : mine;
                const uint32_t best = wave_max_u32(mine);
                int e_win = -1;
#pragma unroll
                for (int c = EC - 1; c >= 0; --c) {
                    const unsigned long long m = __ballot(key[c] == best);
                    if (m != 0ull) e_win = 64 * c + (int)__builtin_ctzll(m);
                }
#pragma unroll
                for (int c = 0; c < EC; ++c)
                    if (lane + 64 * c == e_win) key[c] = 0u;
                win = lane == r ? e_win : win;
                won = lane == r ? best : won;
            }
            if (lane < K) {
                s.ids[i * K + lane] = win;
                s.w[i * K + lane] = ordered_to_float(won);
            }
        }
        __builtin_amdgcn_wave_barrier();
        // lane k < K: the gate weight of slot k
        const float zk = lane < K ? s.w[i * K + lane] : 0.0f;
        const float zmax = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, zk)));
        const float pk = (lane < K) ? expf(zk - zmax) : 0.0f;
        float denom = 0.0f;
        if (p.flags & BM_RENORM_TOPK) {
            for (int k = 0; k < K; ++k)                    // in slot order
                denom += __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, pk), k));
        } else {
            float part = 0.0f;
#pragma unroll
            for (int c = 0; c < EC; ++c) part += (myv[c] == -INFINITY) ? 0.0f : expf(myv[c] - zmax);
            denom = wave_sum(part);
        }
        if (p.flags & BM_PSI_TOKEN) {
            // token-aware buddy priority needs every expert's softmax probability for this token: keep
            // (zmax, 1 / sum over all experts) for the substitution below, or write the probabilities out
            // when the substitution runs in a later kernel
            float part = 0.0f;
#pragma unroll
            for (int c = 0; c < EC; ++c) part += (myv[c] == -INFINITY) ? 0.0f : __expf(myv[c] - zmax);
            const float inv_all = 1.0f / wave_sum(part);
            if (lane == 0) { s.zmax[i] = zmax; s.inv_den[i] = inv_all; }
            if (p.probs_out != nullptr) {
#pragma unroll
                for (int c = 0; c < EC; ++c) {
                    const int e = lane + 64 * c;
                    if (e < E) p.probs_out[(size_t)(t0 + i) * E + e] = __expf(myv[c] - zmax) * inv_all;
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        if (lane < K) {
            p.ids[(size_t)(t0 + i) * K + lane] = s.ids[i * K + lane];
            s.w[i * K + lane] = pk / denom;
        }
    }
    __syncthreads();

    const int n = ntok * K;
    if (p.bitmap == nullptr) {                   // routing only
        for (int idx = tid; idx < n; idx += blockDim.x) p.w[(size_t)t0 * K + idx] = s.w[idx];
        return;
    }

    // stage residency bitmap and buddy table in LDS
    const bool psi_mode = (p.flags & BM_PSI_TOKEN) != 0;         // the logits stay where they are
    const bool tab_in_lds = !psi_mode && E * p.R <= cap_ints;
    int32_t *s_table = reinterpret_cast<int32_t *>(logits);
    if (tab_in_lds)
        for (int idx = tid; idx < E * p.R; idx += blockDim.x) s_table[idx] = p.table[idx];
    for (int idx = tid; idx < BM_MAX_E; idx += blockDim.x) s.counts[idx] = 0;
    if (tid < 4) { s.bitmap[tid] = (tid < ec) ? p.bitmap[tid] : 0ull; s.stats[tid] = 0; s.req[tid] = 0ull; s.dist[tid] = 0; }
    __syncthreads();

    int H = p.H;
    if (p.flags & BM_GATE_DIST) {
        // this tile holds the whole batch (the host guarantees it): set of requested experts, Eq. 2
        for (int idx = tid; idx < n; idx += blockDim.x) {
            const int e = s.ids[idx];
            atomicOr(&s.req[e >> 6], 1ull << (e & 63));
        }
        __syncthreads();
        int n_req = 0, n_cpu = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            n_req += __popcll(s.req[i]);
            n_cpu += __popcll(s.req[i] & ~s.bitmap[i]);
        }
        const bool bypass = dist_bypass(n_req, n_cpu, p.beta);
        if (bypass) H = 0;                       // every miss is dropped
        if (tid == 0) { s.dist[0] = n_req; s.dist[1] = n_cpu; s.dist[2] = bypass ? 1 : 0; }
    }

    const int32_t *tab = tab_in_lds ? s_table : p.table;
    uint64_t resident[EC];
#pragma unroll
    for (int i = 0; i < EC; ++i) resident[i] = s.bitmap[i];
    if ((p.flags & (BM_GATE_ANY | BM_PSI_TOKEN)) || ((p.flags & BM_REMAP_UNIQUE) && K > 1)) {
        // Algorithm 1 proper, with its per-token gates and priorities
        uint32_t *accept = reinterpret_cast<uint32_t *>(s.lut);
        for (int e = tid; e < E; e += blockDim.x) accept[e] = acceptable_entries<EC>(tab + (size_t)e * p.R, H, E, resident);
        __syncthreads();
        PsiSource psi{};
        if (psi_mode) { psi.q = p.q; psi.eta = p.eta; psi.stride = stride; psi.logits = logits; psi.zmax = s.zmax; psi.inv_den = s.inv_den; }
        remap_tile<EC>(ntok, K, E, p.R, p.flags, p.tau, p.gamma, p.rho, resident, accept, tab, s.ids, s.w, s.used, s.stats, psi);
        for (int idx = tid; idx < n; idx += blockDim.x) {
            const int e = s.ids[idx];
            if (e >= 0) atomicAdd(&s.counts[e], 1);
        }
    } else {
        // without the U_t test the substitute depends on the expert alone: one lane per expert looks up its
        // row's first acceptable entry, then every assignment is a table lookup
        for (int e = tid; e < E; e += blockDim.x) {
            const bool res = test_bit<EC>(resident, e);
            const uint32_t m = res ? 0u : acceptable_entries<EC>(tab + (size_t)e * p.R, H, E, resident);
            const int out = res ? e : m != 0u ? tab[(size_t)e * p.R + __builtin_ctz(m)] : -1;
            s.lut[e] = out | (res ? 0 : 0x40000000);       // bit 30 marks "was not resident"
        }
        __syncthreads();
        for (int idx = tid; idx < n; idx += blockDim.x) {
            const int v = s.lut[s.ids[idx]];
            const bool miss = (v & 0x40000000) != 0 || v < 0;
            const int out = v < 0 ? -1 : (v & 0x3fffffff);
            s.ids[idx] = out;
            if (out < 0) s.w[idx] = 0.0f;
            if (miss) atomicAdd(&s.stats[0], 1);
            if (miss && out >= 0) atomicAdd(&s.stats[1], 1);
            if (out < 0) atomicAdd(&s.stats[2], 1);
            if (out >= 0) atomicAdd(&s.counts[out], 1);
        }
    }
    __syncthreads();

    for (int idx = tid; idx < n; idx += blockDim.x) {
        p.ids2[(size_t)t0 * K + idx] = s.ids[idx];
        p.w[(size_t)t0 * K + idx] = s.w[idx];
    }
    // histograms are stored expert-major ([E][tiles]): the single workgroup that scans them reads and writes
    // whole lines, the strided side is spread over the many workgroups here
    const int n_tiles_all = (p.T + p.tile_tokens - 1) / p.tile_tokens;
    for (int e = tid; e < E; e += blockDim.x) p.tile_counts[(size_t)e * n_tiles_all + tile] = s.counts[e];
    if (tid < 3) p.tile_stats[tile * 4 + tid] = s.stats[tid];
}

// ---------------------------------------------------------------------------
// Tail of the front end when one workgroup owns every tile (at most
// FUSED_TILES tiles, i.e. decode-sized batches): group offsets, row-tile table,
// statistics and the stable placement, from the per-tile histograms and
// substituted ids kept in LDS.  Saves the scan and scatter launches.
// ---------------------------------------------------------------------------
constexpr int FUSED_TILES = 1;

struct FusedLds {
    alignas(16) int32_t ids[FUSED_TILES][TILE_T * BM_MAX_K];   // substituted ids of every tile
    int32_t counts[FUSED_TILES][BM_MAX_E];         // per-tile histograms
    int32_t stats[FUSED_TILES][4];
    int32_t dist[4];                               // distribution gate counters (single-tile batches)
    int32_t start[BM_MAX_E + 16];                  // group offsets
    int32_t tstart[BM_MAX_E + 16];                 // first row tile of each group
};

// exclusive prefix sum over the wave; `total` = sum over all lanes.  Four shifts inside each row of 16 lanes, then
// the row sums handed on (DPP moves of a few cycles each; a lane permute through LDS takes over a hundred)
__device__ __forceinline__ int wave_excl_scan(int v, int &total) {
    int incl = v;
#define BM_DPP_ADD(ctrl_, rows_) incl += __builtin_amdgcn_update_dpp(0, incl, ctrl_, rows_, 0xF, false);
    BM_DPP_ADD(0x111, 0xF)     // row_shr 1
    BM_DPP_ADD(0x112, 0xF)     // row_shr 2
    BM_DPP_ADD(0x114, 0xF)     // row_shr 4
    BM_DPP_ADD(0x118, 0xF)     // row_shr 8
    BM_DPP_ADD(0x142, 0xA)     // lane 15 of each row into the next row (rows 1 and 3)
    BM_DPP_ADD(0x143, 0xC)     // lane 31 into rows 2 and 3
#undef BM_DPP_ADD
    total = __builtin_amdgcn_readlane(incl, 63);
    return incl - v;
}

// Per expert, the set of the assignments that hold it: bit a % 64 of masks[e * set_stride(A) + a / 64] for assignment a of
// A whose substituted ids sit in LDS (-1 = dropped).  The number of earlier assignments with the same expert - the rank
// that a stable placement needs - is then a few population counts instead of a walk over the assignments.  Every thread
// of the workgroup calls it; ends with a barrier.
__device__ __forceinline__ void assignment_sets(const int32_t *ids, int A, int E, unsigned long long *masks) {
    const int tid = threadIdx.x, stride = set_stride(A);
    for (int i = tid; i < E * stride; i += blockDim.x) masks[i] = 0ull;
    __syncthreads();
    for (int a = tid; a < A; a += blockDim.x)
        if ((unsigned)ids[a] < (unsigned)E) atomicOr(&masks[ids[a] * stride + (a >> 6)], 1ull << (a & 63));
    __syncthreads();
}
__device__ __forceinline__ int earlier_assignments(const unsigned long long *masks, int A, int e, int a) {
    const unsigned long long *m = masks + e * set_stride(A);
    int rank = __popcll(m[a >> 6] & ((1ull << (a & 63)) - 1ull));
    for (int w = 0; w < (a >> 6); ++w) rank += __popcll(m[w]);
    return rank;
}

// Stable placement: the position of assignment a is start[e] plus its rank in its expert's set.
__device__ __forceinline__ void place_assignments(const int32_t *ids, int A, int E, int K, const int32_t *start,
                                                  const unsigned long long *masks, const ScatterParams &c) {
    for (int a = threadIdx.x; a < A; a += blockDim.x) {
        const int e = ids[a];
        const int pos = (unsigned)e < (unsigned)E ? start[e] + earlier_assignments(masks, A, e, a) : -1;
        if (pos >= 0) {
            c.perm[pos] = a;
            if (c.row_token) c.row_token[pos] = a / K;
        }
        c.inv_perm[a] = pos;
    }
}

// The two row-tile lists of a projection that runs both tile heights in one launch (p.mixed): a group of n rows
// gives n / 256 tiles of 256 rows, and its rest one more of them when it exceeds 128 rows, else (when there is
// a rest) one 128-row tile.  Called by every thread of the workgroup once `start` (G + 1 group starts in LDS)
// is valid; the last wave does the work - scans over the groups in registers, a few consecutive groups per
// lane - while the others go on.
__device__ void write_mixed_tile_tables(const ScanParams &p, const int32_t *start) {
    if (!p.mixed) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if (wave != nw - 1) return;
    const int G = p.E + p.n_shared;
    constexpr int PER = (BM_MAX_E + 8 + 63) / 64;
    int nb[PER], ns[PER], sum_b = 0, sum_s = 0;        // sum_s: 128-row tiles, and live groups from bit 16 on
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int g = lane * PER + i;
        const int n = g < G ? start[g + 1] - start[g] : 0;
        const int rest = n & 255;
        nb[i] = (n >> 8) + (rest > 128 ? 1 : 0);
        ns[i] = (rest >= 1 && rest <= 128) ? 1 : 0;
        sum_b += nb[i];
        sum_s += ns[i] + (n > 0 ? 1 << 16 : 0);
    }
    int tot_b, tot_s;
    int run_b = wave_excl_scan(sum_b, tot_b), run_s = wave_excl_scan(sum_s, tot_s) & 0xffff;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int g = lane * PER + i;
        for (int j = 0; j < nb[i]; ++j) {
            p.mt_group_b[run_b + j] = g;
            p.mt_row0_b[run_b + j] = start[g] + j * 256;
        }
        if (ns[i]) {
            p.mt_group_s[run_s] = g;
            p.mt_row0_s[run_s] = start[g] + nb[i] * 256;
        }
        run_b += nb[i];
        run_s += ns[i];
    }
    if (lane == 0) {
        p.n_mtiles_b[0] = tot_b; p.n_mtiles_b[1] = start[G];
        p.n_mtiles_s[0] = tot_s & 0xffff; p.n_mtiles_s[1] = start[G]; p.n_mtiles_s[2] = tot_s >> 16;
    }
}

// Offsets and the list of row tiles from the group starts in LDS (start: G + 1 rows, tstart: G + 1 tiles);
// every thread of one workgroup calls it.  For the decode projections (largest_first) the list holds the
// live groups by falling row count: a group is one work-item column of their grid, groups with more rows take
// longer per item, and handing the big ones out first leaves the short items for the end of the launch.
__device__ void write_group_tables(const ScanParams &p, const int32_t *start, const int32_t *tstart) {
    const int tid = threadIdx.x, G = p.E + p.n_shared;
    for (int g = tid; g <= G; g += blockDim.x) p.offsets[g] = start[g];
    if (p.largest_first) {
        // eight lanes per group share the comparisons: group h comes first when it has more rows, or as many and a
        // lower index, i.e. when rows * 512 - index is larger (one signed 64-bit difference, no chain of conditions)
        const int part = tid & 7;
        for (int g0 = 0; g0 < G; g0 += blockDim.x >> 3) {
            const int g = min(g0 + (tid >> 3), G - 1);
            const int n = start[g + 1] - start[g];
            const long long mine = (long long)n * 512 - g;
            int rank = 0;
#pragma unroll 4
            for (int h = part; h < G; h += 8) {
                const long long d = mine - ((long long)(start[h + 1] - start[h]) * 512 - h);
                rank += (int)((unsigned long long)d >> 63);
            }
            rank += __shfl_xor(rank, 1, WAVE);
            rank += __shfl_xor(rank, 2, WAVE);
            rank += __shfl_xor(rank, 4, WAVE);
            if (part == 0 && n > 0 && g0 + (tid >> 3) < G) {
                p.mt_group[rank] = g;
                p.mt_row0[rank] = start[g];
            }
        }
    } else {
        for (int g = tid; g < G; g += blockDim.x) {
            const int nt = tstart[g + 1] - tstart[g];
            for (int i = 0; i < nt; ++i) {
                p.mt_group[tstart[g] + i] = g;
                p.mt_row0[tstart[g] + i] = start[g] + i * p.BM;
            }
        }
    }
}

// Everything after the per-expert counts of a batch whose substituted ids sit in LDS (one workgroup):
// group offsets, the list of row tiles (or of live groups, largest first, for the decode projections),
// statistics, stable placement.  counts: E entries in LDS; start / tstart: LDS scratch of G + 1 entries;
// masks: assignment_sets() of the ids; local_stats: the three substitution counters in LDS, or null to add up the
// per-tile ones.  Every thread of the workgroup calls it, after a barrier behind the writes of ids, counts and masks.
__device__ void finish_groups(const ScanParams &p, const ScatterParams &c, const int32_t *ids, int A,
                              const int32_t *counts, int32_t *start, int32_t *tstart, const unsigned long long *masks,
                              const int32_t *local_stats) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int E = p.E, G = p.E + p.n_shared, K = c.K;
    if (wave == 0) {                               // exclusive scans over the groups, a few consecutive groups per lane
        constexpr int PER = (BM_MAX_E + 8 + 63) / 64;
        int cnt[PER], nt[PER], sum_c = 0, sum_t = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int g = lane * PER + i;
            const int n = g < E ? counts[g] : (g < G ? p.T : 0);
            cnt[i] = n;
            nt[i] = (n + p.BM - 1) / p.BM;
            sum_c += n;
            sum_t += nt[i];
        }
        int tot_c, tot_t;
        int run_c = wave_excl_scan(sum_c, tot_c), run_t = wave_excl_scan(sum_t, tot_t);
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int g = lane * PER + i;
            if (g <= G) { start[g] = run_c; tstart[g] = run_t; }
            run_c += cnt[i];
            run_t += nt[i];
        }
        if (lane == 0) { p.n_mtiles[0] = tot_t; p.n_mtiles[1] = tot_c; }
    }
    __syncthreads();
    write_group_tables(p, start, tstart);
    write_mixed_tile_tables(p, start);
    if (p.stats != nullptr && wave < 3) {          // one wave per counter
        int sum = 0;
        if (local_stats != nullptr) sum = local_stats[wave];
        else {
            if (p.tile_stats != nullptr)
                for (int t = lane; t < p.n_tiles; t += WAVE) sum += p.tile_stats[t * 4 + wave];
#pragma unroll
            for (int m = 32; m >= 1; m >>= 1) sum += __shfl_xor(sum, m, WAVE);
        }
        if (lane == 0) { p.stats[wave] = sum; p.stats[3 + wave] = 0; }
    }
    place_assignments(ids, A, E, K, start, masks, c);
    const int live = start[E];
    for (int pos = live + tid; pos < A; pos += blockDim.x) c.perm[pos] = -1;
    if (c.row_token)
        for (int sidx = 0; sidx < p.n_shared; ++sidx)
            for (int t = tid; t < p.T; t += blockDim.x) c.row_token[start[E + sidx] + t] = t;
}

__device__ void fused_tail(const FrontParams &p, FusedLds &fs, int n_tiles, unsigned long long *masks) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int E = p.E, K = p.K, n_shared = p.scan.n_shared, G = E + n_shared, BM = p.scan.BM;
    // group offsets and row-tile starts: one wave, up to 5 consecutive groups per lane
    if (wave == 0) {
        constexpr int PER = (BM_MAX_E + 8 + 63) / 64;
        int cnt[PER], nt[PER], sum_c = 0, sum_t = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int g = lane * PER + i;
            int c = 0;
            if (g < E) { for (int t = 0; t < n_tiles; ++t) c += fs.counts[t][g]; }
            else if (g < G) c = p.T;
            cnt[i] = c;
            nt[i] = (c + BM - 1) / BM;
            sum_c += c;
            sum_t += nt[i];
        }
        int tot_c, tot_t;
        int run_c = wave_excl_scan(sum_c, tot_c), run_t = wave_excl_scan(sum_t, tot_t);
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int g = lane * PER + i;
            if (g <= G) { fs.start[g] = run_c; fs.tstart[g] = run_t; }
            run_c += cnt[i];
            run_t += nt[i];
        }
        if (lane == 0) { p.scan.n_mtiles[0] = tot_t; p.scan.n_mtiles[1] = tot_c; }
    }
    __syncthreads();
    for (int g = tid; g <= G; g += blockDim.x) p.scan.offsets[g] = fs.start[g];
    for (int g = tid; g < G; g += blockDim.x) {
        const int ntile = fs.tstart[g + 1] - fs.tstart[g];
        for (int i = 0; i < ntile; ++i) {
            p.scan.mt_group[fs.tstart[g] + i] = g;
            p.scan.mt_row0[fs.tstart[g] + i] = fs.start[g] + i * BM;
        }
    }
    write_mixed_tile_tables(p.scan, fs.start);
    if (p.scan.stats != nullptr && tid < 3) {
        int sum = 0;
        for (int t = 0; t < n_tiles; ++t) sum += fs.stats[t][tid];
        p.scan.stats[tid] = sum;
        p.scan.stats[3 + tid] = (p.flags & BM_GATE_DIST) ? fs.dist[tid] : 0;
    }
    // stable placement (the batch is one tile)
    const int live = fs.start[E];
    assignment_sets(fs.ids[0], p.T * K, E, masks);
    place_assignments(fs.ids[0], p.T * K, E, K, fs.start, masks, p.scat);
    for (int pos = live + tid; pos < p.T * K; pos += blockDim.x) p.scat.perm[pos] = -1;
    if (p.scat.row_token)
        for (int sidx = 0; sidx < n_shared; ++sidx)
            for (int t = tid; t < p.T; t += blockDim.x) p.scat.row_token[fs.start[E + sidx] + t] = t;
}

// The router product of a token has one order of additions, whatever kernel, batch size or tile it is computed in, so
// that a token's routing does not depend on what else is in the batch or on the call (an engine that fetches the
// experts named by bm_route_topk finds the layer asking for the same ones).  KW waves take every KW-th batch of k-steps
// in turn; their sums w_0 .. w_KW-1 are added as H = partial_tiles<NB, KW, 16>() chains (w_j, w_j+H, w_j+2H, ..), the
// chains by pairs: H is the number of partial tiles (16 tokens x NB * 16 experts) that the front kernels' LDS holds side
// by side.  Tiles of 32 tokens add up their two blocks of 16 one after the other.
template <int NB, int KW, int ROWS>
__host__ __device__ constexpr int partial_tiles() {
    constexpr int fit = (74 * 1024) / (ROWS * (NB * 16 + 4) * 4);
    return fit >= KW ? KW : fit;
}
// v_0 .. v_N-1, `stride` apart: chains of every H-th value, the H chains by pairs
template <int N, int H>
__device__ __forceinline__ float add_slots(const float *at, int stride) {
    static_assert(N % H == 0, "whole chains");
    float v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = at[i * stride];
#pragma unroll
    for (int i = H; i < N; ++i) v[i % H] += v[i];
#pragma unroll
    for (int d = 1; d < H; d *= 2)
#pragma unroll
        for (int i = 0; i + d < H; i += 2 * d) v[i] += v[i + d];
    return v[0];
}

// ---------------------------------------------------------------------------
// bf16 front kernel: router product on MFMA 16x16x32 (tokens x experts),
// operands read from global memory directly in the instruction's layout:
// lane l supplies row/column (l % 16) and the 8 consecutive k values starting
// at 8 * (l / 16), i.e. one 16-byte load per operand per k-step, 64 contiguous
// bytes per row.  (The vector memory path moves one 128-byte line per two
// cycles whatever part of it is used, and with many experts these loads bound
// the kernel; the 32x32x16 form reads 32 bytes per row and instruction.)  The
// waves split the hidden dimension in batches of U k-steps; the loads of a
// batch are all issued before its MFMAs.  The partial logit tiles of the waves
// are written to LDS side by side and added there; when they do not all fit,
// some waves first add into another's tile (one order of additions in any case, see partial_tiles).
// NB = number of 16-expert column blocks, NW = waves per workgroup, NH = parts of the expert blocks over the waves (the
// other factor of NW splits the hidden dimension): 128 experts on 16 waves of 4 blocks each have twice the loads in
// flight and half the tokens to rank per wave that 8 waves of 8 blocks have, in the same registers.
// FUSED: one workgroup walks all (<= FUSED_TILES) tiles and finishes the
// grouping itself.
// ---------------------------------------------------------------------------
template <int NB, int NW, int U, bool FUSED, int NH = 1>
__global__ void __launch_bounds__(NW * 64) front_bf16_kernel(FrontParams p) {
    static_assert(TILE_T == 32, "two 16-token row blocks per tile");
    constexpr int STRIDE = NB * 16 + 4;                  // the four row groups of a partial tile start 16 banks apart
    constexpr int TILE = TILE_T * STRIDE;
    constexpr int NBW = NB / NH, KW = NW / NH;           // expert blocks of a wave, waves along the hidden dimension
    constexpr int NS = partial_tiles<NB, KW, TILE_T>(), NS2 = partial_tiles<NB, KW, 16>();   // kept side by side
    static_assert(NS2 <= 2 * NS, "the partial tiles of 16 tokens fit");
    __shared__ __attribute__((aligned(16))) float part[NS * TILE];
    static_assert(sizeof(part) >= NB * 16 * set_stride(TILE_T * BM_MAX_K) * 8, "holds the assignment sets as well");
    constexpr bool CAN_STAGE = !FUSED && U >= 2 && U % 2 == 0;
    __shared__ u32x4 stage[CAN_STAGE ? NW * 256 : 1];            // 4 KB per wave (see the staged product below)
    __shared__ FrontLds s;
    __shared__ FusedLds fs_store[FUSED ? 1 : 0 + 1];
    FusedLds &fs = fs_store[0];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, kq = lane >> 4;
    const int kw = NH == 1 ? wave : wave % KW, nb0 = NH == 1 ? 0 : wave / KW * NBW;
    const uint16_t *x = static_cast<const uint16_t *>(p.x);
    const uint16_t *wr = static_cast<const uint16_t *>(p.wr);
    const int n_tiles = (p.T + p.tile_tokens - 1) / p.tile_tokens;
    const int tile_begin = FUSED ? 0 : blockIdx.x, tile_end = FUSED ? n_tiles : blockIdx.x + 1;

    const int ksteps = p.d >> 5;
    const int nbatch = ksteps / U;
    static_assert((NW * 64) % (NB * 16) == 0, "a thread adds up logits of one expert only");
    const int my_e = tid % (NB * 16);
    const float my_bias = (p.bias != nullptr && my_e < p.E) ? p.bias[my_e] : 0.0f;

    for (int tile = tile_begin; tile < tile_end; ++tile) {
        const int t0 = tile * p.tile_tokens;
        const bool two = min(p.tile_tokens, p.T - t0) > 16;   // the tile's second 16-token block holds tokens (uniform)
        f32x4 acc[2][NBW];
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb) acc[tb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};

        // Staged product: the operands are fetched as whole 128-byte lines (8 rows per instruction, half as
        // many lines touched as with 64 bytes per row - and with many experts the lines touched bound the
        // kernel) and turned into the MFMA operand order through a wave-private LDS area of two 2 KB
        // blocks: stored 8 rows x 128 bytes per register, read back 16 rows x 16 bytes per fragment, the
        // 16-byte pieces of a row rotated by the row index against bank conflicts.  The blocks are reused
        // operand block after operand block; no barrier: only the writing wave touches its area, and a
        // wave's LDS operations stay in order.  A batch is LPB lines (two k-steps each) of every operand.
        // (not in the fused kernel, which has no registers to spare: it serves batches of a few tokens,
        // whose direct loads touch few lines anyway; not with 256 experts, whose batch would not fit)
        const bool staged = CAN_STAGE;
        int ks_done = nbatch * U;                                      // k-steps covered by the batched loops
        const bool given = !FUSED && p.logits != nullptr;              // the product is there already
        if (given) {
            ks_done = ksteps;
        } else if (CAN_STAGE) {
            constexpr int LPB = U / 2 > 0 ? U / 2 : 1;
            u32x4 *area = stage + (CAN_STAGE ? wave : 0) * 256;       // [block 0..1][row 0..15][piece 0..7]
            const int lrow = lane >> 3, lpiece = lane & 7;
            const uint16_t *xs_[2][2];
            int woff[NBW][2], wslot[2], rslot[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int r = 8 * j + lrow;
#pragma unroll
                for (int tb = 0; tb < 2; ++tb) xs_[tb][j] = x + (size_t)min(t0 + tb * 16 + r, p.T - 1) * p.d + lpiece * 8;
#pragma unroll
                for (int nb = 0; nb < NBW; ++nb) woff[nb][j] = min((nb0 + nb) * 16 + r, p.E - 1) * p.d + lpiece * 8;
                wslot[j] = r * 8 + (lpiece ^ (r & 7));
                rslot[j] = r16 * 8 + ((j * 4 + kq) ^ (r16 & 7));     // fragment of the line's k-step j
            }
            const int nlb = p.d / (64 * LPB);
            ks_done = nlb * 2 * LPB;
            for (int bt = kw; bt < nlb; bt += KW) {
                const int k0 = bt * 64 * LPB;
                u32x4 rx[LPB][2][2], rw[LPB][NBW][2];                   // [line][operand block][row group]
#pragma unroll
                for (int h = 0; h < LPB; ++h)
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        rx[h][0][j] = ldg128(xs_[0][j] + k0 + h * 64);
                        if (two) rx[h][1][j] = ldg128(xs_[1][j] + k0 + h * 64);
#pragma unroll
                        for (int nb = 0; nb < NBW; ++nb) rw[h][nb][j] = ldg128(wr + woff[nb][j] + k0 + h * 64);
                    }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int h = 0; h < LPB; ++h) {
                    bf16x8 fa[2][2];
#pragma unroll
                    for (int tb = 0; tb < 2; ++tb) {
                        if (tb == 1 && !two) break;
#pragma unroll
                        for (int j = 0; j < 2; ++j) area[tb * 128 + wslot[j]] = rx[h][tb][j];
#pragma unroll
                        for (int ks = 0; ks < 2; ++ks) fa[tb][ks] = as_bf16x8(area[tb * 128 + rslot[ks]]);
                    }
#pragma unroll
                    for (int nb = 0; nb < NBW; ++nb) {
                        u32x4 *ar = area + (nb & 1) * 128;
#pragma unroll
                        for (int j = 0; j < 2; ++j) ar[wslot[j]] = rw[h][nb][j];
#pragma unroll
                        for (int ks = 0; ks < 2; ++ks) {
                            const bf16x8 b = as_bf16x8(ar[rslot[ks]]);
                            acc[0][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[0][ks], b, acc[0][nb], 0, 0, 0);
                            if (two)
                                acc[1][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[1][ks], b, acc[1][nb], 0, 0, 0);
                        }
                    }
                }
            }
        }
        // operand rows of the direct loads (set up behind the staged product, which has no registers to spare for them)
        const uint16_t *xa[2], *wb[NBW];
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) xa[tb] = x + (size_t)min(t0 + tb * 16 + r16, p.T - 1) * p.d + kq * 8;
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb) wb[nb] = wr + (size_t)min((nb0 + nb) * 16 + r16, p.E - 1) * p.d + kq * 8;
        for (int bt = kw; !staged && !given && bt < nbatch; bt += KW) {
            const int k0 = bt * U * 32;
            u32x4 ra[2][U], rb[NBW][U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                ra[0][u] = ldg128(xa[0] + k0 + u * 32);
                if (two) ra[1][u] = ldg128(xa[1] + k0 + u * 32);
#pragma unroll
                for (int nb = 0; nb < NBW; ++nb) rb[nb][u] = ldg128(wb[nb] + k0 + u * 32);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int nb = 0; nb < NBW; ++nb) {
                    acc[0][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(ra[0][u]), as_bf16x8(rb[nb][u]), acc[0][nb], 0, 0, 0);
                    if (two)
                        acc[1][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(ra[1][u]), as_bf16x8(rb[nb][u]), acc[1][nb], 0, 0, 0);
                }
        }
        for (int ks = ks_done + kw; ks < ksteps; ks += KW) {          // k-steps past the last full batch
            const bf16x8 a0 = as_bf16x8(ldg128(xa[0] + ks * 32)), a1 = as_bf16x8(ldg128(xa[1] + ks * 32));
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb) {
                const bf16x8 b = as_bf16x8(ldg128(wb[nb] + ks * 32));
                acc[0][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, b, acc[0][nb], 0, 0, 0);
                acc[1][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, b, acc[1][nb], 0, 0, 0);
            }
        }

        // D[i][j] of a 16x16 block: lane holds column j = l % 16 and rows i = 4 * (l / 16) + v.
        // Partial tiles of 16 tokens sit side by side in LDS; wave w of an expert part adds into slot w % NS2 in round
        // w / NS2, then the slots are added: one fixed association, reproducible.
        constexpr int STEP = NW * 64 / (NB * 16), ROWS_PER = (16 + STEP - 1) / STEP;   // rows a sweep of the threads adds up
        const int my_i = tid / (NB * 16);
        if (given) {
            const int n = min(p.tile_tokens, p.T - t0) * p.E;
            for (int idx = tid; idx < n; idx += NW * 64) {
                const int i = idx / p.E, e = idx - i * p.E;
                part[i * STRIDE + e] = p.logits[(size_t)t0 * p.E + idx];
            }
        } else {
            float sum[2][ROWS_PER];
            constexpr bool BOTH = NS == KW;              // the waves' tiles of 32 tokens fit side by side: both blocks at once
            constexpr int SLOT = BOTH ? TILE : 16 * STRIDE, ROUNDS = (KW + NS2 - 1) / NS2;
#pragma unroll
            for (int tb = 0; tb < 2; ++tb) {
                if (tb == 1 && !two) break;
                if (tb == 1 && !BOTH) __syncthreads();   // the first block's slots have been read
#pragma unroll
                for (int r = 0; r < ROUNDS; ++r) {
                    if (kw / NS2 == r) {
                        float *mine = part + (kw % NS2) * SLOT + (BOTH ? tb * 16 * STRIDE : 0);
#pragma unroll
                        for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                float *q = &mine[(4 * kq + v) * STRIDE + (nb0 + nb) * 16 + r16];
                                *q = (r == 0 ? 0.0f : *q) + acc[tb][nb][v];
                            }
                    }
                    if (!BOTH) __syncthreads();
                }
                if (BOTH) continue;
#pragma unroll
                for (int j = 0; j < ROWS_PER; ++j)
                    if (my_i + j * STEP < 16)
                        sum[tb][j] = add_slots<NS2, NS2>(part + (my_i + j * STEP) * STRIDE + my_e, SLOT) + my_bias;
            }
            if (BOTH) {
                __syncthreads();
#pragma unroll
                for (int tb = 0; tb < 2; ++tb)
#pragma unroll
                    for (int j = 0; j < ROWS_PER; ++j)
                        if ((tb == 0 || two) && my_i + j * STEP < 16)
                            sum[tb][j] = add_slots<NS2, NS2>(part + (tb * 16 + my_i + j * STEP) * STRIDE + my_e, SLOT) + my_bias;
            }
            // the first two slots become the logit tile (a thread writes only where it alone has read)
#pragma unroll
            for (int tb = 0; tb < 2; ++tb) {
                if (tb == 1 && !two) break;
#pragma unroll
                for (int j = 0; j < ROWS_PER; ++j)
                    if (my_i + j * STEP < 16) part[(tb * 16 + my_i + j * STEP) * STRIDE + my_e] = sum[tb][j];
            }
        }
        __syncthreads();
        tile_epilogue<(NB + 3) / 4>(p, part, STRIDE, TILE, s, tile);
        if (FUSED) {
            __syncthreads();
            const int n = min(p.tile_tokens, p.T - t0) * p.K;
            for (int idx = tid; idx < n; idx += NW * 64) fs.ids[tile][idx] = s.ids[idx];
            for (int e = tid; e < p.E; e += NW * 64) fs.counts[tile][e] = s.counts[e];
            if (tid < 3) { fs.stats[tile][tid] = s.stats[tid]; fs.dist[tid] = s.dist[tid]; }
            __syncthreads();
        }
    }
    if (FUSED) fused_tail(p, fs, n_tiles, reinterpret_cast<unsigned long long *>(part));
    // a batch of one tile: this workgroup holds every substituted id and the histogram, and finishes the
    // grouping itself instead of leaving it to a launch of its own
    if (!FUSED && p.tail) {
        __syncthreads();
        unsigned long long *masks = reinterpret_cast<unsigned long long *>(part);    // the logits and the table are done
        assignment_sets(s.ids, p.T * p.K, p.E, masks);
        finish_groups(p.scan, p.scat, s.ids, p.T * p.K, s.counts, fs.start, fs.tstart, masks, s.stats);
    }
}

// ---------------------------------------------------------------------------
// The router product in a launch of its own, for few tiles and many experts: the front kernels have one workgroup per
// 16 tokens, which reads the whole router matrix through one unit (bf16, 128 experts: 8 of 18 us) and, in fp32,
// multiplies 16 x 128 x 2048 on it (14 us of matrix instructions, plus the sums between them).  Here a workgroup
// takes 16 tokens x 16 experts, its 8 waves split the hidden dimension; the front kernel then starts from the
// logits.  Same operand layouts, k-step batches and order of additions as there, so the same bits.  Qwen3-shaped layer:
// fp32, 128 tokens 48 us -> 11 + 10 us; bf16, 8 tokens 17 us -> 5 + 10 us.
// ---------------------------------------------------------------------------
constexpr int ROUTER_NW = 8;

// NB: the front kernel's expert blocks, whose k-step batches (32 values, 16 with 256 experts) and sum order this takes
// (8 serves 33 to 128 experts: 4 and 8 blocks are the same in both)
static_assert(partial_tiles<4, ROUTER_NW, 16>() == partial_tiles<8, ROUTER_NW, 16>(), "one instantiation for both");
template <int NB>
__global__ void __launch_bounds__(ROUTER_NW * 64) router_f32_kernel(FrontParams p) {
    __shared__ f32x4 part[ROUTER_NW][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r16 = lane & 15, quad = lane >> 4;
    const int e0 = blockIdx.x * 16, t0 = blockIdx.y * 16, d = p.d;
    const float *xr = static_cast<const float *>(p.x) + (size_t)min(t0 + r16, p.T - 1) * d + quad * 4;
    const float *wr = static_cast<const float *>(p.wr) + (size_t)min(e0 + r16, p.E - 1) * d + quad * 4;
    constexpr int KS = NB <= 8 ? 2 : 1, G = 2 / KS, KB = KS * 16, STEP = ROUTER_NW * KB;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int k = wave * KB; k < d; k += G * STEP) {               // (d is a multiple of 32)
        f32x4 a[G][KS], b[G][KS];
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const int at = min(k + g * STEP, d - KB) + s * 16;
                a[g][s] = *(const BM_GLOBAL f32x4 *)(xr + at);
                b[g][s] = *(const BM_GLOBAL f32x4 *)(wr + at);
            }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (g > 0 && k + g * STEP >= d) break;
            f32x4 c[KS];
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                f32x4 q[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) q[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[g][s][i], b[g][s][i], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                c[s] = (q[0] + q[1]) + (q[2] + q[3]);
            }
            acc += KS == 2 ? c[0] + c[KS - 1] : c[0];
        }
    }
    part[wave][lane] = acc;
    __syncthreads();
    if (wave != 0) return;
    f32x4 sum;
#pragma unroll
    for (int v = 0; v < 4; ++v)
        sum[v] = add_slots<ROUTER_NW, partial_tiles<NB, ROUTER_NW, 16>()>(reinterpret_cast<const float *>(part) + lane * 4 + v, 64 * 4);
    const int e = e0 + r16;
    if (e >= p.E) return;
    const float bias = p.bias != nullptr ? p.bias[e] : 0.0f;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int t = t0 + 4 * quad + v;
        if (t < p.T) p.logits[(size_t)t * p.E + e] = sum[v] + bias;
    }
}

// NB as above: batches of two k-steps of 32, of one with 256 experts; a wave has eight k-steps in flight
template <int NB>
__global__ void __launch_bounds__(ROUTER_NW * 64) router_bf16_kernel(FrontParams p) {
    __shared__ f32x4 part[ROUTER_NW][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r16 = lane & 15, kq = lane >> 4;
    const int e0 = blockIdx.x * 16, t0 = blockIdx.y * 16, ksteps = p.d >> 5;
    const uint16_t *xr = static_cast<const uint16_t *>(p.x) + (size_t)min(t0 + r16, p.T - 1) * p.d + kq * 8;
    const uint16_t *wr = static_cast<const uint16_t *>(p.wr) + (size_t)min(e0 + r16, p.E - 1) * p.d + kq * 8;
    constexpr int U = NB <= 8 ? 2 : 1, G = 8 / U;
    const int nbatch = ksteps / U;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    int bt = wave;
    for (; bt + (G - 1) * ROUTER_NW < nbatch; bt += G * ROUTER_NW) {
        u32x4 a[G][U], b[G][U];
        const uint16_t *xk = xr + bt * (U * 32), *wk = wr + bt * (U * 32);
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                a[g][u] = ldg128(xk + (g * ROUTER_NW * U + u) * 32);
                b[g][u] = ldg128(wk + (g * ROUTER_NW * U + u) * 32);
            }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int u = 0; u < U; ++u) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a[g][u]), as_bf16x8(b[g][u]), acc, 0, 0, 0);
    }
    for (; bt < nbatch; bt += ROUTER_NW)                   // the batches past the last full group
#pragma unroll
        for (int u = 0; u < U; ++u)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(ldg128(xr + (bt * U + u) * 32)), as_bf16x8(ldg128(wr + (bt * U + u) * 32)), acc, 0, 0, 0);
    for (int ks = nbatch * U + wave; ks < ksteps; ks += ROUTER_NW)     // a k-step past the last full batch
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(ldg128(xr + ks * 32)), as_bf16x8(ldg128(wr + ks * 32)), acc, 0, 0, 0);
    part[wave][lane] = acc;
    __syncthreads();
    if (wave != 0) return;
    f32x4 sum;
#pragma unroll
    for (int v = 0; v < 4; ++v)
        sum[v] = add_slots<ROUTER_NW, partial_tiles<NB, ROUTER_NW, 16>()>(reinterpret_cast<const float *>(part) + lane * 4 + v, 64 * 4);
    const int e = e0 + r16;
    if (e >= p.E) return;
    const float bias = p.bias != nullptr ? p.bias[e] : 0.0f;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int t = t0 + 4 * kq + v;
        if (t < p.T) p.logits[(size_t)t * p.E + e] = sum[v] + bias;
    }
}

// fp32: from 33 experts on, up to 64 tiles (a quarter of the units), whole 32-value batches of aligned rows only.
// bf16: from 65 experts on, up to 64 tokens (the layer at 1 / 8 / 32 / 64 / 128 / 2048 tokens, 128 experts, us:
// 40.0 58.2 80.3 97.6 124.8 259 with the product in the front kernel, 37.6 56.3 79.2 96.7 124.6 266 on its own;
// 64 experts at 1 / 8 / 32 tokens: 49.2 66.1 90.0 | 49.2 66.6 89.5).
bool front_wants_logits(const FrontParams &p, int dtype) {
    return dtype == BM_F32 ? p.E > 32 && p.T <= 1024 && p.d % 32 == 0 && aligned16(p.x) && aligned16(p.wr) : p.E > 64 && p.T <= 64;
}

// ---------------------------------------------------------------------------
// fp32 front kernel: 16 tokens per workgroup, router product (tokens x experts) on v_mfma_f32_16x16x4_f32.
// Lane l loads four consecutive k of row / column l % 16 (one 16-byte piece, piece l / 16 of a 16-wide k
// slice); MFMA i of the slice takes component i of every piece, the same k order for both operands.  The
// waves split the hidden dimension in batches of 32 and load a batch ahead; a batch is summed as a
// tree over its MFMAs and added to the wave's sum, the waves' sums are added in wave order (no rounding chain is
// longer than the lane-strided sums of the kernel it replaces).  Bound by the matrix instruction with many experts
// (16 x 128 x 2048: 14 us on one unit) and by latency with few.  It replaces one dot product per wave at a time:
// Qwen3-shaped layer, 128 tokens 4354 us; tiny layer (8 experts, d = 64) 22 us.
// NB = number of 16-expert column blocks, NW = waves, KS = 16-wide k slices per batch, PRE: load a batch ahead.
// ---------------------------------------------------------------------------
template <int NB, int NW, int KS, bool PRE, int NH = 1>
__global__ void __launch_bounds__(NW * 64) front_f32_kernel(FrontParams p) {
    constexpr int TT = 16, STRIDE = NB * 16 + 4, TILE = TT * STRIDE;
    constexpr int NBW = NB / NH, KW = NW / NH;           // as in the bf16 kernel
    constexpr int NS = partial_tiles<NB, KW, TT>();      // kept side by side
    __shared__ __attribute__((aligned(16))) float part[NS * TILE];
    static_assert(sizeof(part) >= NB * 16 * set_stride(TT * BM_MAX_K) * 8, "holds the assignment sets as well");
    __shared__ FrontLds s;
    __shared__ int32_t start[BM_MAX_E + 16], tstart[BM_MAX_E + 16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r16 = lane & 15, quad = lane >> 4;
    const int tile = blockIdx.x, t0 = tile * TT, d = p.d;
    const float *xr = static_cast<const float *>(p.x) + (size_t)min(t0 + r16, p.T - 1) * d;
    const int kw = NH == 1 ? wave : wave % KW, nb0 = NH == 1 ? 0 : wave / KW * NBW;
    const float *wr[NBW];
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb) wr[nb] = static_cast<const float *>(p.wr) + (size_t)min((nb0 + nb) * 16 + r16, p.E - 1) * d;

    f32x4 acc[NBW];
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    constexpr int KB = KS * 16;
    const int nbatch = p.logits != nullptr ? 0 : (d + KB - 1) / KB;       // the product is there already
    const bool aligned = (d & 3) == 0 && aligned16(p.x) && aligned16(p.wr);    // rows start on 16-byte boundaries
    f32x4 a[2][KS], b[2][NBW][KS];
    auto load = [&](int bt, f32x4 (&ra)[KS], f32x4 (&rb)[NBW][KS]) {
        const bool plain = aligned && (bt + 1) * KB <= d;         // uniform
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int k = bt * KB + ks * 16 + quad * 4;
            if (plain) {
                ra[ks] = *(const BM_GLOBAL f32x4 *)(xr + k);
#pragma unroll
                for (int nb = 0; nb < NBW; ++nb) rb[nb][ks] = *(const BM_GLOBAL f32x4 *)(wr[nb] + k);
            } else {                                              // past the end: zeros in both operands
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool in = k + i < d;
                    const int kc = in ? k + i : 0;
                    ra[ks][i] = in ? xr[kc] : 0.0f;
#pragma unroll
                    for (int nb = 0; nb < NBW; ++nb) rb[nb][ks][i] = in ? wr[nb][kc] : 0.0f;
                }
            }
        }
    };
    auto multiply = [&](const f32x4 (&ra)[KS], const f32x4 (&rb)[NBW][KS]) {
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb) {
            f32x4 c[KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                f32x4 q[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    q[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(ra[ks][i], rb[nb][ks][i], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                c[ks] = (q[0] + q[1]) + (q[2] + q[3]);
            }
            acc[nb] += KS == 2 ? c[0] + c[KS - 1] : c[0];
        }
    };
    if (PRE) {
        if (kw < nbatch) load(kw, a[0], b[0]);
        for (int bt = kw; bt < nbatch; bt += 2 * KW) {
            if (bt + KW < nbatch) load(bt + KW, a[1], b[1]);
            multiply(a[0], b[0]);
            if (bt + KW >= nbatch) break;
            if (bt + 2 * KW < nbatch) load(bt + 2 * KW, a[0], b[0]);
            multiply(a[1], b[1]);
        }
    } else {
        for (int bt = kw; bt < nbatch; bt += KW) {
            load(bt, a[0], b[0]);
            multiply(a[0], b[0]);
        }
    }
    if (p.logits != nullptr) {
        const int n = min(TT, p.T - t0) * p.E;
        for (int idx = tid; idx < n; idx += NW * 64) {
            const int i = idx / p.E, e = idx - i * p.E;
            part[i * STRIDE + e] = p.logits[(size_t)t0 * p.E + idx];
        }
    } else {
        // D of a 16x16 block: lane holds column (expert) r16 and rows (tokens) 4 * quad + v; slots as in the bf16 kernel
        for (int r = 0; r < (KW + NS - 1) / NS; ++r) {
            if (kw / NS == r) {
                float *mine = part + (kw % NS) * TILE;
#pragma unroll
                for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        float *q = &mine[(4 * quad + v) * STRIDE + (nb0 + nb) * 16 + r16];
                        *q = (r == 0 ? 0.0f : *q) + acc[nb][v];
                    }
            }
            __syncthreads();
        }
        for (int idx = tid; idx < TT * NB * 16; idx += NW * 64) {
            const int i = idx / (NB * 16), e = idx - i * (NB * 16);
            part[i * STRIDE + e] = add_slots<NS, NS>(part + i * STRIDE + e, TILE) + ((p.bias != nullptr && e < p.E) ? p.bias[e] : 0.0f);
        }
    }
    __syncthreads();
    tile_epilogue<(NB + 3) / 4>(p, part, STRIDE, NS * TILE, s, tile);
    if (p.tail) {
        __syncthreads();
        unsigned long long *masks = reinterpret_cast<unsigned long long *>(part);    // the logits and the table are done
        assignment_sets(s.ids, p.T * p.K, p.E, masks);
        finish_groups(p.scan, p.scat, s.ids, p.T * p.K, s.counts, start, tstart, masks, s.stats);
    }
}

// ---------------------------------------------------------------------------
// Stand-alone substitution kernel: tiles of 64 tokens; table, acceptable entries and ids in LDS.  Bound by latency.
// With the distribution gate every workgroup reads all routed ids for the request set (no scratch memory, no
// grid-wide wait): 16 bytes per load, eight loads in flight per lane (3001 tokens of 8 out of 128 experts: 8.8 us; 62 us
// with one 4-byte load in flight, the buddy rows scanned entry by entry and a whole walk per lane).
// A single workgroup stores the counters, several add theirs to zeros (launch_remap).
// ---------------------------------------------------------------------------
template <int W, int KC = 0>        // KC = 1: one slot per token, else p.K
__global__ void __launch_bounds__(1024) remap_kernel(RemapParams p) {
    extern __shared__ int32_t s_table[];                // E * R entries, then E acceptable-entry masks
    __shared__ int32_t s_req[64 * W];                   // distribution gate: the expert was routed to
    __shared__ int32_t s_ids[REMAP_TOK * BM_MAX_K];
    __shared__ unsigned long long s_used[REMAP_TOK * W];
    __shared__ int32_t s_stats[3];
    const int tid = threadIdx.x;
    const int ec = (p.E + 63) >> 6;
    uint32_t *accept = reinterpret_cast<uint32_t *>(s_table + p.E * p.R);
    if ((int)blockIdx.x * REMAP_TOK < p.T) {           // the first tile's ids along with the table
        const int n0 = min(REMAP_TOK, p.T - (int)blockIdx.x * REMAP_TOK) * p.K;
        for (int idx = tid; idx < n0; idx += blockDim.x) s_ids[idx] = p.ids_in[(size_t)blockIdx.x * REMAP_TOK * p.K + idx];
    }
    for (int idx = tid; idx < p.E * p.R; idx += blockDim.x) s_table[idx] = p.table[idx];
    uint64_t resident[W];
#pragma unroll
    for (int i = 0; i < W; ++i) resident[i] = i < ec ? p.bitmap[i] : 0ull;
    for (int e = tid; e < 64 * W; e += blockDim.x) s_req[e] = 0;
    if (tid < 3) s_stats[tid] = 0;
    __syncthreads();
    int H = p.H;
    if (p.flags & BM_GATE_DIST) {
        // Eq. 2 over the whole batch; every lane that meets an expert stores the same 1
        const size_t n = (size_t)p.T * p.K, n_vec = aligned16(p.ids_in) ? n >> 2 : 0;     // others one by one
        typedef __attribute__((ext_vector_type(4))) int32_t i32x4;
        for (size_t v0 = tid; v0 < n_vec; v0 += 8 * (size_t)blockDim.x) {
            i32x4 v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const size_t at = v0 + i * (size_t)blockDim.x;
                v[i] = at < n_vec ? *(const BM_GLOBAL i32x4 *)(p.ids_in + 4 * at) : i32x4{-1, -1, -1, -1};
            }
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if ((unsigned)v[i][c] < (unsigned)p.E) s_req[v[i][c]] = 1;
        }
        for (size_t a = 4 * n_vec + tid; a < n; a += blockDim.x) {
            const int e = p.ids_in[a];
            if ((unsigned)e < (unsigned)p.E) s_req[e] = 1;
        }
        __syncthreads();
        int n_req = 0, n_cpu = 0;
#pragma unroll
        for (int i = 0; i < W; ++i) {
            const uint64_t req = __ballot(s_req[64 * i + (tid & 63)] != 0);
            n_req += __popcll(req);
            n_cpu += __popcll(req & ~resident[i]);
        }
        const bool bypass = dist_bypass(n_req, n_cpu, p.beta);
        if (bypass) H = 0;
        if (p.stats != nullptr && blockIdx.x == 0 && tid == 0) {
            p.stats[3] = n_req; p.stats[4] = n_cpu; p.stats[5] = bypass ? 1 : 0;
        }
    } else if (p.stats != nullptr && blockIdx.x == 0 && tid < 3) {
        p.stats[3 + tid] = 0;
    }
    for (int e = tid; e < p.E; e += blockDim.x) accept[e] = acceptable_entries<W>(s_table + e * p.R, H, p.E, resident);
    __syncthreads();
    for (int t0 = blockIdx.x * REMAP_TOK; t0 < p.T; t0 += gridDim.x * REMAP_TOK) {
        const int ntok = min(REMAP_TOK, p.T - t0), n = ntok * p.K;
        const int32_t *in = p.ids_in + (size_t)t0 * p.K;
        if (t0 != (int)blockIdx.x * REMAP_TOK) {
            for (int idx = tid; idx < n; idx += blockDim.x) s_ids[idx] = in[idx];
            __syncthreads();
        }
        PsiSource psi{};
        if (p.flags & BM_PSI_TOKEN) { psi.q = p.q; psi.eta = p.eta; psi.stride = p.E; psi.probs = p.probs + (size_t)t0 * p.E; }
        remap_tile<W, KC>(ntok, p.K, p.E, p.R, p.flags, p.tau, p.gamma, p.rho, resident, accept, s_table, s_ids,
                      p.w != nullptr ? p.w + (size_t)t0 * p.K : nullptr, s_used, s_stats, psi);
        for (int idx = tid; idx < n; idx += blockDim.x) p.ids_out[(size_t)t0 * p.K + idx] = s_ids[idx];
        __syncthreads();
    }
    if (p.stats != nullptr && tid < 3) {
        if (gridDim.x == 1) p.stats[tid] = s_stats[tid];
        else if (s_stats[tid]) atomicAdd(&p.stats[tid], s_stats[tid]);
    }
}

__global__ void zero_ints_kernel(int32_t *p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

// Per-tile histogram of given ids (stand-alone grouping entry point).
__global__ void __launch_bounds__(256) count_kernel(const int32_t *ids, int T, int K, int E, int tile_tokens,
                                                    int32_t *tile_counts) {
    __shared__ int32_t counts[BM_MAX_E];
    const int tid = threadIdx.x, tile = blockIdx.x, t0 = tile * tile_tokens;
    const int n = min(tile_tokens, T - t0) * K;
    for (int e = tid; e < E; e += blockDim.x) counts[e] = 0;
    __syncthreads();
    for (int idx = tid; idx < n; idx += blockDim.x) {
        const int e = ids[(size_t)t0 * K + idx];
        if ((unsigned)e < (unsigned)E) atomicAdd(&counts[e], 1);
    }
    __syncthreads();
    const int n_tiles_all = (T + tile_tokens - 1) / tile_tokens;
    for (int e = tid; e < E; e += blockDim.x) tile_counts[(size_t)e * n_tiles_all + tile] = counts[e];
}

// ---------------------------------------------------------------------------
// One-workgroup scan: tile histograms -> per-tile bases (relative to the
// group start), group offsets (routed experts, then shared experts with T
// rows each), the row-tile table of the grouped GEMMs, and the summed
// substitution statistics.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(1024) scan_kernel(ScanParams p) {
    __shared__ int32_t total[BM_MAX_E + 8];
    __shared__ int32_t start[BM_MAX_E + 9];
    __shared__ int32_t tstart[BM_MAX_E + 9];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = blockDim.x >> 6;
    const int G = p.E + p.n_shared;
    // per expert: exclusive scan of its counts over the tiles, 64 tiles per wave step.  A wave takes EB
    // experts at a time and issues the loads of SB steps of each together: every load is a round trip
    // to memory, the scans between them are short.
    constexpr int SB = 4, EB = 4;
    for (int e0 = wave; e0 < p.E; e0 += nw * EB) {          // experts e0, e0 + nw, ..: few experts spread over the waves
        int run[EB];
#pragma unroll
        for (int j = 0; j < EB; ++j) run[j] = 0;
        for (int tb = 0; tb < p.n_tiles; tb += SB * WAVE) {
            int c[EB][SB];
#pragma unroll
            for (int j = 0; j < EB; ++j)
#pragma unroll
                for (int i = 0; i < SB; ++i) {
                    const int t = tb + i * WAVE + lane;
                    c[j][i] = (e0 + j * nw < p.E && t < p.n_tiles) ? p.tile_counts[(size_t)(e0 + j * nw) * p.n_tiles + t] : 0;
                }
#pragma unroll
            for (int j = 0; j < EB; ++j)
#pragma unroll
                for (int i = 0; i < SB; ++i) {
                    if (tb + i * WAVE >= p.n_tiles || e0 + j * nw >= p.E) continue;   // uniform over the wave
                    const int t = tb + i * WAVE + lane;
                    int tot;
                    const int ex = wave_excl_scan(c[j][i], tot);
                    if (e0 + j * nw < p.E && t < p.n_tiles) p.tile_base[(size_t)(e0 + j * nw) * p.n_tiles + t] = run[j] + ex;
                    run[j] += tot;
                }
        }
#pragma unroll
        for (int j = 0; j < EB; ++j)
            if (lane == 0 && e0 + j * nw < p.E) total[e0 + j * nw] = run[j];
    }
    for (int g = p.E + tid; g < G; g += blockDim.x) total[g] = p.T;
    __syncthreads();
    if (wave == 0) {                               // exclusive scans over the groups, a few consecutive groups per lane
        constexpr int PER = (BM_MAX_E + 8 + 63) / 64;
        int cnt[PER], nt[PER], sum_c = 0, sum_t = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int g = lane * PER + i;
            const int c = g < G ? total[g] : 0;
            cnt[i] = c;
            nt[i] = (c + p.BM - 1) / p.BM;
            sum_c += c;
            sum_t += nt[i];
        }
        int tot_c, tot_t;
        int run_c = wave_excl_scan(sum_c, tot_c), run_t = wave_excl_scan(sum_t, tot_t);
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int g = lane * PER + i;
            if (g <= G) { start[g] = run_c; tstart[g] = run_t; }
            run_c += cnt[i];
            run_t += nt[i];
        }
        if (lane == 0) { p.n_mtiles[0] = tot_t; p.n_mtiles[1] = tot_c; }
    }
    __syncthreads();
    write_group_tables(p, start, tstart);
    write_mixed_tile_tables(p, start);
    if (p.stats != nullptr && wave < 3) {          // one wave per counter, lanes over the tiles
        int sum = 0;
        if (p.tile_stats != nullptr)
            for (int t = lane; t < p.n_tiles; t += WAVE) sum += p.tile_stats[t * 4 + wave];
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) sum += __shfl_xor(sum, m, WAVE);
        if (lane == 0) { p.stats[wave] = sum; p.stats[3 + wave] = 0; }
    }
}

// ---------------------------------------------------------------------------
// Scatter: position of assignment a = offsets[e] + base of its tile + number
// of earlier assignments of the tile with the same expert.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) scatter_kernel(ScatterParams p) {
    __shared__ int32_t s_ids[TILE_T * BM_MAX_K];
    __shared__ unsigned long long masks[BM_MAX_E * set_stride(TILE_T * BM_MAX_K)];
    const int tid = threadIdx.x, tile = blockIdx.x, t0 = tile * p.tile_tokens;
    const int n_tiles_all = (p.T + p.tile_tokens - 1) / p.tile_tokens;
    const int K = p.K, E = p.E;
    const int ntok = min(p.tile_tokens, p.T - t0);
    const int n = ntok * K;
    for (int idx = tid; idx < n; idx += blockDim.x) {
        const int e = p.ids[(size_t)t0 * K + idx];
        s_ids[idx] = ((unsigned)e < (unsigned)E) ? e : -1;
    }
    assignment_sets(s_ids, n, E, masks);                 // (its first barrier is behind the stores above)
    const int live = p.offsets[E];
    for (int idx = tid; idx < n; idx += blockDim.x) {
        const int e = s_ids[idx];
        const int a = t0 * K + idx;
        int pos = -1;
        if (e >= 0) {
            pos = p.offsets[e] + p.tile_base[(size_t)e * n_tiles_all + tile] + earlier_assignments(masks, n, e, idx);
            p.perm[pos] = a;
            if (p.row_token) p.row_token[pos] = a / K;
        }
        p.inv_perm[a] = pos;
    }
    // positions past the live count hold -1
    for (int idx = tid; idx < p.tile_tokens * K; idx += blockDim.x) {
        const int pos = t0 * K + idx;
        if (pos >= live && pos < p.T * K) p.perm[pos] = -1;
    }
    // rows of the shared experts map to their own token
    if (p.row_token)
        for (int sidx = 0; sidx < p.n_shared; ++sidx) {
            const int base = p.offsets[E + sidx];
            for (int i = tid; i < ntok; i += blockDim.x) p.row_token[base + t0 + i] = t0 + i;
        }
}

// ---------------------------------------------------------------------------
// Scan and scatter in one launch for batches whose histogram (experts x tiles)
// is small enough for every workgroup to sum it by itself: the workgroup of a
// tile adds up, per expert, all tiles (group size) and the tiles before its
// own (its base inside the group) - a wave per expert, lanes over the tiles,
// the loads of EB experts going out together - scans the group sizes, and
// places its assignments.  The workgroup of tile 0 also writes the offsets,
// the row-tile table and the statistics.  Saves the one-workgroup scan launch,
// a chain of dependent round trips to memory (11 us for 64-128 experts).
// ---------------------------------------------------------------------------
constexpr long long TILE_SUM_MAX = 32768;          // histogram entries every workgroup re-reads (128 KB)

__global__ void __launch_bounds__(1024) group_tiles_kernel(ScanParams p, ScatterParams c) {
    __shared__ int32_t total[BM_MAX_E + 8];
    __shared__ int32_t before[BM_MAX_E];
    __shared__ int32_t start[BM_MAX_E + 9];
    __shared__ int32_t tstart[BM_MAX_E + 9];
    __shared__ int32_t s_ids[TILE_T * BM_MAX_K];
    __shared__ unsigned long long masks[BM_MAX_E * set_stride(TILE_T * BM_MAX_K)];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = blockDim.x >> 6;
    const int tile = blockIdx.x, t0 = tile * c.tile_tokens;
    const int K = c.K, E = p.E, G = p.E + p.n_shared;
    const int ntok = min(c.tile_tokens, c.T - t0);
    const int n = ntok * K;
    for (int idx = tid; idx < n; idx += blockDim.x) {
        const int e = c.ids[(size_t)t0 * K + idx];
        s_ids[idx] = ((unsigned)e < (unsigned)E) ? e : -1;
    }
    assignment_sets(s_ids, n, E, masks);                  // (its first barrier is behind the stores above)
    constexpr int EB = 8, SB = 4;                         // every load is a round trip to memory: EB * SB go out together
    for (int e0 = wave; e0 < E; e0 += nw * EB) {          // experts e0, e0 + nw, ..
        int tot[EB], bef[EB];
#pragma unroll
        for (int j = 0; j < EB; ++j) tot[j] = bef[j] = 0;
        for (int tb = 0; tb < p.n_tiles; tb += SB * WAVE) {
            int cnt[EB][SB];
#pragma unroll
            for (int j = 0; j < EB; ++j)
#pragma unroll
                for (int i = 0; i < SB; ++i) {
                    const int t = tb + i * WAVE + lane;
                    cnt[j][i] = (e0 + j * nw < E && t < p.n_tiles) ? p.tile_counts[(size_t)(e0 + j * nw) * p.n_tiles + t] : 0;
                }
#pragma unroll
            for (int j = 0; j < EB; ++j)
#pragma unroll
                for (int i = 0; i < SB; ++i) {
                    tot[j] += cnt[j][i];
                    bef[j] += tb + i * WAVE + lane < tile ? cnt[j][i] : 0;
                }
        }
#pragma unroll
        for (int j = 0; j < EB; ++j) {
            int t, b;                                     // sums over the wave (DPP moves, not lane permutes)
            wave_excl_scan(tot[j], t);
            wave_excl_scan(bef[j], b);
            if (lane == 0 && e0 + j * nw < E) { total[e0 + j * nw] = t; before[e0 + j * nw] = b; }
        }
    }
    for (int g = E + tid; g < G; g += blockDim.x) total[g] = p.T;
    __syncthreads();
    if (wave == 0) {                               // exclusive scans over the groups, a few consecutive groups per lane
        constexpr int PER = (BM_MAX_E + 8 + 63) / 64;
        int cnt[PER], nt[PER], sum_c = 0, sum_t = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int g = lane * PER + i;
            const int cg = g < G ? total[g] : 0;
            cnt[i] = cg;
            nt[i] = (cg + p.BM - 1) / p.BM;
            sum_c += cg;
            sum_t += nt[i];
        }
        int tot_c, tot_t;
        int run_c = wave_excl_scan(sum_c, tot_c), run_t = wave_excl_scan(sum_t, tot_t);
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int g = lane * PER + i;
            if (g <= G) { start[g] = run_c; tstart[g] = run_t; }
            run_c += cnt[i];
            run_t += nt[i];
        }
        if (tile == 0 && lane == 0) { p.n_mtiles[0] = tot_t; p.n_mtiles[1] = tot_c; }
    }
    __syncthreads();
    if (tile == 0) {
        write_group_tables(p, start, tstart);
        write_mixed_tile_tables(p, start);
        if (p.stats != nullptr && wave >= nw - 3) {    // one wave per counter, lanes over the tiles
            const int k = wave - (nw - 3);
            int sum = 0;
            if (p.tile_stats != nullptr)
                for (int t = lane; t < p.n_tiles; t += WAVE) sum += p.tile_stats[t * 4 + k];
#pragma unroll
            for (int m = 32; m >= 1; m >>= 1) sum += __shfl_xor(sum, m, WAVE);
            if (lane == 0) { p.stats[k] = sum; p.stats[3 + k] = 0; }
        }
    }
    // placement: group start + the tile's base inside the group + earlier assignments of the tile with the same expert
    const int live = start[E];
    for (int idx = tid; idx < n; idx += blockDim.x) {
        const int e = s_ids[idx];
        const int a = t0 * K + idx;
        int pos = -1;
        if (e >= 0) {
            pos = start[e] + before[e] + earlier_assignments(masks, n, e, idx);
            c.perm[pos] = a;
            if (c.row_token) c.row_token[pos] = a / K;
        }
        c.inv_perm[a] = pos;
    }
    for (int idx = tid; idx < c.tile_tokens * K; idx += blockDim.x) {      // positions past the live count hold -1
        const int pos = t0 * K + idx;
        if (pos >= live && pos < c.T * K) c.perm[pos] = -1;
    }
    if (c.row_token)                                                         // rows of the shared experts map to their own token
        for (int sidx = 0; sidx < c.n_shared; ++sidx)
            for (int i = tid; i < ntok; i += blockDim.x) c.row_token[start[E + sidx] + t0 + i] = t0 + i;
}

// ---------------------------------------------------------------------------
// Scan and scatter in one workgroup for small batches
// (grouping_small): the substituted ids are staged in LDS, every expert's count
// and the stable positions come from its assignment set.
// Writes what scan_kernel and scatter_kernel write, except the per-tile bases.
// ---------------------------------------------------------------------------
constexpr int SMALL_ANY = 1024, SMALL_A = 2048, SMALL_SETS = 32768;     // see grouping_small

__global__ void __launch_bounds__(1024) group_small_kernel(ScanParams p, ScatterParams c) {
    __shared__ int32_t ids[SMALL_A];
    __shared__ unsigned long long masks[set_stride(SMALL_ANY) * BM_MAX_E];
    static_assert(set_stride(SMALL_ANY) * BM_MAX_E >= SMALL_SETS / 64 + 2 * (SMALL_SETS / SMALL_ANY), "holds the larger batches' sets, rounded up per expert");
    __shared__ int32_t total[BM_MAX_E + 8];
    __shared__ int32_t start[BM_MAX_E + 9];
    __shared__ int32_t tstart[BM_MAX_E + 9];
    const int tid = threadIdx.x, E = p.E, A = c.T * c.K, words = (A + 63) >> 6, stride = set_stride(A);
    for (int a = tid; a < A; a += blockDim.x) {
        const int e = c.ids[a];
        ids[a] = ((unsigned)e < (unsigned)E) ? e : -1;
    }
    assignment_sets(ids, A, E, masks);                   // (its first barrier is behind the stores above)
    for (int e = tid; e < E; e += blockDim.x) {
        int cnt = 0;
        for (int w = 0; w < words; ++w) cnt += __popcll(masks[e * stride + w]);
        total[e] = cnt;
    }
    __syncthreads();
    finish_groups(p, c, ids, A, total, start, tstart, masks, nullptr);
}

// ---------------------------------------------------------------------------
// Host-side launchers
// ---------------------------------------------------------------------------
template <int NB, int NW, int U, int NH = 1>
static void launch_front_bf16(const FrontParams &p, int n_tiles, hipStream_t st) {
    // (the fused tail has no registers to spare for more waves)
    if (p.fused) hipLaunchKernelGGL((front_bf16_kernel<NB, NW / NH, U, true>), dim3(1), dim3(NW / NH * 64), 0, st, p);
    else hipLaunchKernelGGL((front_bf16_kernel<NB, NW, U, false, NH>), dim3(n_tiles), dim3(NW * 64), 0, st, p);
}

// One workgroup for the whole front end (router to placement): only with the distribution gate and a
// batch of at most one tile - the gate's in-tile form needs the whole batch in one workgroup and saves two
// launches.  Otherwise workgroups of 16 tokens plus the grouping kernel are faster at every batch size
// (front end at 1 / 8 / 16 tokens: 13.8 / 13.6 / 14.2 us against 15.0 / 16.0 / 17.7 us); a batch of one such
// workgroup finishes the grouping itself (FrontParams::tail).
bool front_can_fuse(int T, int dtype, uint32_t flags) {
    return dtype == BM_BF16 && (flags & BM_GATE_DIST) && T > 0 && T <= TILE_T;
}

// Tokens per workgroup of the bf16 front kernel (and per tile of the histograms that the scan and scatter
// kernels work on).  A tile's router product is bound by the number of cache lines its loads touch, so
// as long as 32-token tiles would not give every compute unit a workgroup, the batch is cut into 16-token
// tiles on twice the units (measured at 64 tokens: front kernel 12 us instead of 18).
int front_tile_tokens(int T, int dtype, bool fused) {
    if (dtype == BM_F32) return 16;                // one row block of the fp32 matrix instruction
    return (!fused && (T + TILE_T - 1) / TILE_T < 256) ? 16 : TILE_T;
}

int launch_front(const FrontParams &p, int dtype, hipStream_t st) {
    const int n_tiles = (p.T + p.tile_tokens - 1) / p.tile_tokens;
    if (n_tiles == 0) return 0;
    const int nb = (p.E + 15) / 16;
    if (dtype == BM_F32) {
        if (p.logits != nullptr) {
            const dim3 grid(nb, (p.T + 15) / 16), block(ROUTER_NW * 64);
            if (nb <= 8) hipLaunchKernelGGL(router_f32_kernel<8>, grid, block, 0, st, p);
            else hipLaunchKernelGGL(router_f32_kernel<16>, grid, block, 0, st, p);
        }
        if (nb <= 1) hipLaunchKernelGGL((front_f32_kernel<1, 16, 2, true>), dim3(n_tiles), dim3(1024), 0, st, p);
        else if (nb <= 2) hipLaunchKernelGGL((front_f32_kernel<2, 8, 2, true>), dim3(n_tiles), dim3(512), 0, st, p);
        else if (nb <= 4) hipLaunchKernelGGL((front_f32_kernel<4, 8, 2, true>), dim3(n_tiles), dim3(512), 0, st, p);
        else if (nb <= 8) hipLaunchKernelGGL((front_f32_kernel<8, 16, 2, false, 2>), dim3(n_tiles), dim3(1024), 0, st, p);
        else hipLaunchKernelGGL((front_f32_kernel<16, 8, 1, false>), dim3(n_tiles), dim3(512), 0, st, p);
    } else {
        if (p.logits != nullptr) {
            const dim3 grid(nb, (p.T + 15) / 16), block(ROUTER_NW * 64);
            if (nb <= 8) hipLaunchKernelGGL(router_bf16_kernel<8>, grid, block, 0, st, p);
            else hipLaunchKernelGGL(router_bf16_kernel<16>, grid, block, 0, st, p);
        }
        // a tile is latency-bound: 16 waves split the product and rank two tokens each; U keeps a batch
        // of loads ((2 + NB) * U registers quadruples) inside the 128 registers a wave of 16 has
        if (nb <= 1) launch_front_bf16<1, 16, 4>(p, n_tiles, st);
        else if (nb <= 2) launch_front_bf16<2, 16, 4>(p, n_tiles, st);
        else if (nb <= 4) launch_front_bf16<4, 16, 2>(p, n_tiles, st);
        else if (nb <= 8) launch_front_bf16<8, 16, 2, 2>(p, n_tiles, st);
        else launch_front_bf16<16, 8, 1>(p, n_tiles, st);
    }
    return launch_status(__func__);
}

int launch_remap(const RemapParams &p, hipStream_t st) {
    if (p.T <= 0) {
        if (p.stats) hipLaunchKernelGGL(zero_ints_kernel, dim3(1), dim3(64), 0, st, p.stats, 6);
        return launch_status(__func__);
    }
    const size_t lds = (size_t)p.E * (p.R + 1) * sizeof(int32_t);
    // with the distribution gate every workgroup reads all ids for the request set: large workgroups, not too many
    const bool dist = (p.flags & BM_GATE_DIST) != 0;
    const int threads = dist ? 1024 : 256;
    int blocks = 1;
    // in place behind the gate, a single workgroup reads the request set before it overwrites anything
    if (p.T > remap_one_workgroup_tokens(p.K, p.flags) && !(dist && p.ids_out == p.ids_in)) {
        blocks = (p.T - 1) / REMAP_TOK + 1;
        blocks = blocks > (dist ? 256 : 1024) ? (dist ? 256 : 1024) : blocks;
        if (p.stats) hipLaunchKernelGGL(zero_ints_kernel, dim3(1), dim3(64), 0, st, p.stats, 3);
    }
#define BM_REMAP(W_)                                                                                           \
    {                                                                                                          \
        if (p.K == 1) hipLaunchKernelGGL((remap_kernel<W_, 1>), dim3(blocks), dim3(threads), lds, st, p);      \
        else hipLaunchKernelGGL((remap_kernel<W_>), dim3(blocks), dim3(threads), lds, st, p);                  \
    }
    if (p.E <= 64) BM_REMAP(1)
    else if (p.E <= 128) BM_REMAP(2)
    else BM_REMAP(4)
#undef BM_REMAP
    return launch_status(__func__);
}

int launch_count(const int32_t *ids, int T, int K, int E, int tile_tokens, int32_t *tile_counts, hipStream_t st) {
    const int n_tiles = (T + tile_tokens - 1) / tile_tokens;
    if (n_tiles) hipLaunchKernelGGL(count_kernel, dim3(n_tiles), dim3(256), 0, st, ids, T, K, E, tile_tokens, tile_counts);
    return launch_status(__func__);
}

int launch_scan(const ScanParams &p, hipStream_t st) {
    hipLaunchKernelGGL(scan_kernel, dim3(1), dim3(1024), 0, st, p);
    return launch_status(__func__);
}

// The one-workgroup kernel takes up to 1024 assignments, one per thread, whatever the number of experts, and up to 2048 of
// few experts; beyond, a thread's rank adds up too many words.  One workgroup | per-tile histograms and the kernel that
// sums them, us: bm_permute_by_expert (which has to count first in the second form) of 128 experts, 512 / 1024
// assignments 4.1 4.7 | 8.7 8.7, 8 experts, 1536 / 2048 5.4 6.3 | 8.0 8.0; small layers (whose front kernel has counted) of
// 128 experts, 1024 / 2048 assignments 33.7 38.0 | 35.1 37.2, 8 experts, 1536 / 2048 / 4096 45.2 46.3 52.8 | 45.7 46.0 47.4.
bool grouping_small(long long assignments, int E) {
    return assignments <= SMALL_ANY || (assignments <= SMALL_A && assignments * E <= SMALL_SETS);
}

// scan + scatter: one kernel for small batches and for small histograms
int launch_grouping(const ScanParams &sp, const ScatterParams &cp, hipStream_t st) {
    if (grouping_small((long long)cp.T * cp.K, cp.E)) {
        hipLaunchKernelGGL(group_small_kernel, dim3(1), dim3(1024), 0, st, sp, cp);   // also for an empty batch: offsets
        return launch_status(__func__);
    }
    const int n_tiles = (cp.T + cp.tile_tokens - 1) / cp.tile_tokens;
    if ((long long)sp.E * n_tiles <= TILE_SUM_MAX) {
        hipLaunchKernelGGL(group_tiles_kernel, dim3(n_tiles), dim3(1024), 0, st, sp, cp);
        return launch_status(__func__);
    }
    const int rc = launch_scan(sp, st);
    return rc | launch_scatter(cp, st);
}

int launch_scatter(const ScatterParams &p, hipStream_t st) {
    const int n_tiles = (p.T + p.tile_tokens - 1) / p.tile_tokens;
    if (n_tiles) hipLaunchKernelGGL(scatter_kernel, dim3(n_tiles), dim3(256), 0, st, p);
    return launch_status(__func__);
}

}  // namespace bm
