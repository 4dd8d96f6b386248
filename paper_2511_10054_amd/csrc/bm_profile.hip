// Profiling statistics and buddy-list construction on the device.
//
//   coact_kernel        per-expert activation counts A and pairwise co-activation counts M of a batch
//                       of routed ids, added to running totals
//   buddy_build_kernel  per pivot: peers ranked by conditional co-activation, cut at the cumulative
//                       frequency threshold
//
// Both are exact integer work up to one fp64 comparison per list entry.
#include "bm_dispatch_rules.h"
#include "bm_kernels.h"

namespace bm {

// Co-activation counts by bit sets.  A workgroup takes CO_TOK tokens and CO_ROWS pivots: it writes, per expert, the
// set of its chunk's tokens that hold the expert (one bit per token, LDS atomic OR - an expert listed twice sets one
// bit twice, ids out of range set none; neighbouring lanes own different words, so that a popular expert's bits do
// not queue on one), then counts every pair (pivot i, expert j) as the population count of
// the two sets' intersection and adds it to the global int64 totals; the pair (i, i) is the activation count.
// Bound by latency: one read of the chunk's ids, two barriers, the LDS reads of a thread's pairs (4 pivots: 5.8 us for
// 4096 tokens of 8 out of 128 experts).  The kernel it
// replaces walked a token per wave with lane permutes and flushed a whole triangle every 64 tokens: 41 us.
// CO_TOK = 512 halves the chain of a workgroup (sets to clear, bits to set that meet in a bank, words of a pair to count) and
// doubles the additions to the totals; which it takes: coact_short_chunks.
constexpr int CO_ROWS = 4;

template <int CO_TOK>
__global__ void __launch_bounds__(CO_TOK) coact_kernel(const int32_t *ids, int T, int K, int E, unsigned long long *A,
                                                       unsigned long long *M) {
    constexpr int CO_WORDS = CO_TOK / 64;
    __shared__ unsigned long long bits[BM_MAX_E][CO_WORDS + 1];         // padded: rows start in different banks
    constexpr int PAIRS = CO_ROWS * BM_MAX_E / CO_TOK;                  // pairs of a thread
    const int tid = threadIdx.x, row0 = blockIdx.x * CO_ROWS;
    const int n_pairs = min(CO_ROWS, E - row0) * E;
    const int chunks = T / CO_TOK + (T % CO_TOK ? 1 : 0);
    int n[PAIRS] = {};
    for (int c = blockIdx.y; c < chunks; c += gridDim.y) {
        const bool mine = tid < T - c * CO_TOK;
        const int32_t *row = ids + ((size_t)c * CO_TOK + tid) * K;
        int e[8];                                                       // eight loads in flight, the first ones while
#pragma unroll                                                          // the sets are cleared
        for (int i = 0; i < 8; ++i) e[i] = mine && i < K ? row[i] : -1;
        for (int i = tid; i < E * (CO_WORDS + 1); i += CO_TOK) (&bits[0][0])[i] = 0ull;
        __syncthreads();
        for (int k0 = 0; k0 < K; k0 += 8) {
            if (k0 > 0) {
#pragma unroll
                for (int i = 0; i < 8; ++i) e[i] = mine && k0 + i < K ? row[k0 + i] : -1;
            }
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if ((unsigned)e[i] < (unsigned)E)
                    atomicOr(reinterpret_cast<unsigned *>(bits[e[i]]) + tid % (2 * CO_WORDS), 1u << tid / (2 * CO_WORDS));
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < PAIRS; ++q) {
            const int idx = tid + q * CO_TOK;
            if (idx >= n_pairs) break;
            const unsigned long long *bi = bits[row0 + idx / E], *bj = bits[idx % E];
#pragma unroll
            for (int w = 0; w < CO_WORDS; ++w) n[q] += __popcll(bi[w] & bj[w]);
        }
        __syncthreads();                                                // the next chunk clears the sets
    }
#pragma unroll
    for (int q = 0; q < PAIRS; ++q) {
        const int idx = tid + q * CO_TOK;
        if (idx >= n_pairs) break;
        const int i = row0 + idx / E, j = idx % E;
        if (n[q]) atomicAdd(i == j ? &A[i] : &M[(size_t)i * E + j], (unsigned long long)n[q]);
    }
}

// One workgroup per pivot i, thread j owns peer j.  A peer's rank is the number of peers with a larger count, or the
// same count and a lower index (the order of q = count / row sum); peers of rank r form the sequence pi_i.  The
// first wave then scans the prefix sums, four ranks per lane: the list ends at the first t with
//   count(pi_i(1..t)) >= alpha * row sum         (one fp64 product, one comparison)
// cut to at most R entries, at least one if the row sum is positive.  Bound by latency: E broadcast reads of the
// counts per thread (one wave ranking two experts per lane and lane 0 walking the prefix sums: 14 us for 128 experts).
__global__ void __launch_bounds__(BM_MAX_E) buddy_build_kernel(const long long *M, int E, int R, float alpha,
                                                               int32_t *table, int32_t *list_len, float *q_out) {
    __shared__ long long s_cnt[BM_MAX_E];
    __shared__ int32_t s_order[BM_MAX_E];
    const int i = blockIdx.x, j = threadIdx.x;
    const long long mine = (j < E && j != i) ? M[(size_t)i * E + j] : 0;
    s_cnt[j] = mine;
    s_order[j] = -1;
    __syncthreads();
    if (mine > 0) {
        int rank = 0;
#pragma unroll 16
        for (int o = 0; o < E; ++o) {
            const long long co = s_cnt[o];
            rank += (int)(co > mine) | ((int)(co == mine) & (int)(o < j));
        }
        s_order[rank] = j;
    }
    __syncthreads();
    if (j >= WAVE) return;
    constexpr int PER = BM_MAX_E / WAVE;
    int ord[PER];
    long long cnt[PER], own = 0, total = 0;
#pragma unroll
    for (int c = 0; c < PER; ++c) {
        ord[c] = s_order[j * PER + c];
        cnt[c] = ord[c] >= 0 ? s_cnt[ord[c]] : 0;
        own += cnt[c];
        total += s_cnt[j * PER + c];
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) total += __shfl_xor(total, m, WAVE);
    long long cum = own;                             // inclusive scan of the listed counts over the lanes
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1) {
        const long long o = __shfl_up(cum, d, WAVE);
        if (j >= d) cum += o;
    }
    cum -= own;
    const double need = (double)alpha * (double)total;
    int reach = E;                                   // first rank of this lane whose prefix sum reaches the threshold
    int listed = 0;
#pragma unroll
    for (int c = 0; c < PER; ++c) {
        cum += cnt[c];
        if (ord[c] >= 0) {
            ++listed;
            if ((double)cum >= need && reach == E) reach = j * PER + c;
        }
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        reach = min(reach, __shfl_xor(reach, m, WAVE));
        listed += __shfl_xor(listed, m, WAVE);
    }
    const int t_i = min(min(reach + 1, listed), R);
    for (int r = j; r < R; r += WAVE) {
        const int o = r < t_i ? s_order[r] : -1;
        table[(size_t)i * R + r] = o;
        if (q_out) q_out[(size_t)i * R + r] = o >= 0 ? (float)((double)s_cnt[o] / (double)total) : 0.0f;
    }
    if (j == 0 && list_len) list_len[i] = t_i;
}

int launch_coactivation(const int32_t *ids, int T, int K, int E, long long *A, long long *M, hipStream_t st) {
    if (T > 0) {
        // up to two workgroups per unit (four of the short ones); those of a longer batch walk several chunks before they
        // add their counts up
        const bool brief = coact_short_chunks(T, K, E);
        const int tok = brief ? 512 : 1024, rows = (E + CO_ROWS - 1) / CO_ROWS;
        const int chunks = T / tok + (T % tok ? 1 : 0), most = 512 * 1024 / tok / rows;
        const dim3 grid(rows, chunks < most ? chunks : most);
        unsigned long long *a = reinterpret_cast<unsigned long long *>(A), *m = reinterpret_cast<unsigned long long *>(M);
        if (brief) hipLaunchKernelGGL(coact_kernel<512>, grid, dim3(512), 0, st, ids, T, K, E, a, m);
        else hipLaunchKernelGGL(coact_kernel<1024>, grid, dim3(1024), 0, st, ids, T, K, E, a, m);
    }
    return launch_status(__func__);
}

int launch_buddy_build(const long long *M, int E, int R, float alpha, int32_t *table, int32_t *list_len, float *q,
                       hipStream_t st) {
    hipLaunchKernelGGL(buddy_build_kernel, dim3(E), dim3(BM_MAX_E), 0, st, M, E, R, alpha, table, list_len, q);
    return launch_status(__func__);
}

}  // namespace bm
