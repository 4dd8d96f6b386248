// fp32 expert projections: grouped tiles on the fp32 matrix instruction, and a row-by-row fallback for
// widths the tiles cannot load.
#include "bm_kernels.h"

namespace bm {

__device__ __forceinline__ float silu_precise(float a) { return a / (1.0f + expf(-a)); }

// group of a row: offsets is non-decreasing with G+1 entries
__device__ __forceinline__ int find_group(const int32_t *offsets, int G, int pos) {
    int lo = 0, hi = G;               // offsets[lo] <= pos < offsets[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (offsets[mid] <= pos) lo = mid; else hi = mid;
    }
    return lo;
}

template <bool DUAL>
__global__ void __launch_bounds__(256) rowwise_f32_kernel(GemmParams p) {
    extern __shared__ float s_row[];
    __shared__ int s_g;
    const int pos = blockIdx.x;
    if (pos >= p.n_mtiles[1]) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) s_g = find_group(p.offsets, p.n_groups, pos);
    const int src = p.row_map ? p.row_map[pos] : pos;
    const float *arow = static_cast<const float *>(p.a) + (size_t)src * p.Kd;
    for (int j = tid; j < p.Kd; j += blockDim.x) s_row[j] = arow[j];
    __syncthreads();
    const int g = s_g;
    const float *b0 = (g < p.E) ? static_cast<const float *>(p.b0) + (size_t)g * p.N * p.Kd
                                : static_cast<const float *>(p.sb0) + (size_t)(g - p.E) * p.N * p.Kd;
    const float *b1 = nullptr;
    if (DUAL)
        b1 = (g < p.E) ? static_cast<const float *>(p.b1) + (size_t)g * p.N * p.Kd
                       : static_cast<const float *>(p.sb1) + (size_t)(g - p.E) * p.N * p.Kd;
    float *c = static_cast<float *>(p.c) + (size_t)pos * p.N;
    for (int n = wave; n < p.N; n += 4) {
        const float *r0 = b0 + (size_t)n * p.Kd;
        float s0 = 0.0f, s1 = 0.0f;
        if (DUAL) {
            const float *r1 = b1 + (size_t)n * p.Kd;
            for (int j = lane; j < p.Kd; j += WAVE) {
                s0 = fmaf(r0[j], s_row[j], s0);
                s1 = fmaf(r1[j], s_row[j], s1);
            }
            s0 = wave_sum(s0);
            s1 = wave_sum(s1);
            if (lane == 0) c[n] = silu_precise(s0) * s1;
        } else {
            for (int j = lane; j < p.Kd; j += WAVE) s0 = fmaf(r0[j], s_row[j], s0);
            s0 = wave_sum(s0);
            if (lane == 0) c[n] = s0;
        }
    }
}

// ---------------------------------------------------------------------------
// Grouped fp32 tiles: up to 64 rows of one group x 64 weight rows per workgroup (DUAL: 32 of W_gate and the same
// 32 of W_up), on v_mfma_f32_16x16x4_f32 (exact fp32 products and sums; the fp32 matrix rate is that of the
// vector FMA units, but an operand is read from LDS once per 16 x 16 block instead of once per product).
//
// What bounds it: groups of at most ~30 rows are bound by streaming their weights once, larger ones by the fp32
// matrix rate.  The kernel it replaces (one workgroup per row, each wave a weight row at a time) read an expert's
// weights once per ROW: 2790 + 2630 us for the two projections of the Qwen3-shaped layer at 128 tokens; here 123 to 148 + 75 to 85 us by inputs
// (floors 90 and 48: 599 and 322 MB read at 6.7 TB/s).  Groups of a few rows, which stream, and groups of tens of rows,
// which multiply, take turns on a unit.
//
//  - Weights are the first MFMA operand, activations the second: a lane ends up with four consecutive output
//    columns of one row (16-byte stores).  The four waves are two blocks of 16 weight rows (of each half of the
//    64) times the two 16-wide halves of a k-step; the halves meet in LDS at the end.  16-row blocks past the end
//    of the group are not multiplied (NBT = 1, 2 or 4 blocks, chosen per tile).
//  - k-steps of 32 values = one 128-byte line per row, fetched straight into LDS as whole lines
//    (global_load_lds_dwordx4, 8 rows per instruction) into a ring of F32_STAGES stages; row r's 16-byte piece p
//    sits at slot p ^ ((r >> 1) & 7) (applied by choosing which piece a lane fetches): conflict-free ds_read_b128.
//    A piece is four consecutive k; the four MFMAs of a 16-wide k slice take component 0, 1, 2, 3 of every lane's
//    piece, i.e. k in the order {0,4,8,12}, {1,5,9,13}, .. - the same order for both operands.
//  - One wait and one barrier per k-step: stage kt has landed for every wave, and everybody is done reading stage
//    kt - 1, whose slot takes the loads of stage kt + F32_STAGES - 1.
//  - The sum over k is a tree: CHAIN MFMAs of four values in a row, the rest of a 16-wide slice by pairs, eight
//    k-steps, the other k-steps, the two halves.  One MFMA chain over 2048 values would round that many times in a
//    row; this way no level is longer than the chains of the kernel it replaces (Kd / 64 values per lane and a tree
//    over the lanes), and the error against 64 bits is no larger.  Short reductions, where that tree was most of
//    the sum, take CHAIN = 1; from 1024 on CHAIN = 2 spares a third of the additions.
//  - Weights of a group that one row tile covers are not read again: they are loaded non-temporally (AUX = 2; unless the
//    memory-side cache holds the weights of all live groups until the layer's next call), and the units
//    of an XCD enter the reduction at 32 different places and walk it as a circle (rot; the tree's shape stays): weight
//    rows lie a multiple of 4 KB apart in many layers, and workgroups in step all ask the same memory channels.
//    Qwen3-shaped layer at 16 tokens 76 + 42 -> 64 + 38 us, DeepSeek-shaped at 8 tokens 74 + 30 -> 59 + 27.
//  - Three waves a SIMD are asked for, not left to happen: with room for more registers the compiler puts the MFMA results
//    into accumulator registers and copies each of them out for the tree, as many instructions as the tree itself
//    (8 experts of 256 rows, d = 2048, F = 4096: 783 + 401 -> 718 + 367 us; Qwen3-shaped at 128 tokens 143 + 90 -> 127 + 78).
// Needs Kd % 32 == 0.
// ---------------------------------------------------------------------------
#define BM_LDS __attribute__((address_space(3)))
constexpr int F32_ROWS = 64;            // activation rows per tile
constexpr int F32_STAGES = 3;           // 48 KB: three workgroups per unit (4 or 5 stages leave two: gate/up 162 / 164 us against 150)
constexpr int F32_CHUNKS = 8;           // row tiles of a group that run side by side

template <bool DUAL, int NBT, int CHAIN, int AUX>
__device__ __forceinline__ void f32_tile(const GemmParams &p, float *smem, const float *b0, const float *b1,
                                         int row0, int row_end, int n0, int rot) {
    constexpr int S = F32_STAGES;
    constexpr int AROWS = 16 * NBT;
    constexpr int STAGE = (AROWS + 64) * 32;                     // floats
    constexpr int NA = NBT >= 2 ? NBT / 2 : 1;                   // activation loads per wave and stage
    constexpr int NL = NA + 2;                                   // loads per wave and stage
    constexpr int BLK = DUAL ? 32 : 64;                          // output columns of the tile
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r16 = lane & 15, quad = lane >> 4;
    const int wn = wave >> 1, ks = wave & 1;                     // block of 16 weight rows, half of the k-step
    const int N = p.N, Kd = p.Kd, KT = Kd >> 5;

    // load instruction: 8 rows x 128 bytes; lane i fetches row i / 8 and the piece that belongs into slot i % 8
    const float *pa[NA], *pb[2];
    int la[NA];
#pragma unroll
    for (int j = 0; j < NA; ++j) {
        const int blk = NBT >= 2 ? wave + 4 * j : (wave & 1);    // one 16-row block: two waves repeat the others' loads
        const int r = blk * 8 + (lane >> 3);
        const int pos = min(row0 + r, row_end - 1);
        const int src = p.row_map ? ldg_i32(p.row_map + pos) : pos;
        pa[j] = static_cast<const float *>(p.a) + (size_t)src * Kd + (((lane & 7) ^ ((r >> 1) & 7)) << 2);
        la[j] = blk * 256;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {                                // rows 0-31 and 32-63 of the weight part
        const int r = wave * 8 + (lane >> 3);
        const int n = min(n0 + r + (DUAL ? 0 : 32 * j), N - 1);
        pb[j] = (DUAL && j ? b1 : b0) + (size_t)n * Kd + (((lane & 7) ^ ((r >> 1) & 7)) << 2);
    }
#define BM_F32_LOAD(kt_, slot_)                                                                               \
    {                                                                                                         \
        const int kr_ = min((kt_), KT - 1) + rot;                                                             \
        const int k_ = (kr_ >= KT ? kr_ - KT : kr_) * 32;                                                     \
        float *st_ = smem + (slot_) * STAGE;                                                                  \
        _Pragma("unroll") for (int j = 0; j < 2; ++j)                                                         \
            __builtin_amdgcn_global_load_lds((const BM_GLOBAL void *)(pb[j] + k_),                            \
                (BM_LDS void *)(st_ + (AROWS + j * 32 + wave * 8) * 32), 16, 0, AUX);                         \
        _Pragma("unroll") for (int j = 0; j < NA; ++j)                                                        \
            __builtin_amdgcn_global_load_lds((const BM_GLOBAL void *)(pa[j] + k_),                            \
                                             (BM_LDS void *)(st_ + la[j]), 16, 0, 0);                         \
    }
    // fragment offset inside 16 rows of a stage
    const int foff = r16 * 32 + (((4 * ks + quad) ^ ((r16 >> 1) & 7)) << 2);
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 sum[2][NBT], mid[2][NBT];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int tb = 0; tb < NBT; ++tb) sum[m][tb] = mid[m][tb] = zero;

#pragma unroll
    for (int st = 0; st < S - 1; ++st) BM_F32_LOAD(st, st);
    int cur = 0, wr = S - 1;
    for (int kt = 0; kt < KT; ++kt) {
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"((S - 2) * NL) : "memory");
        BM_F32_LOAD(kt + S - 1, wr);
        const float *st = smem + cur * STAGE;
        f32x4 w[2], x[NBT];
#pragma unroll
        for (int m = 0; m < 2; ++m) w[m] = *reinterpret_cast<const f32x4 *>(st + (AROWS + m * 32 + wn * 16) * 32 + foff);
#pragma unroll
        for (int tb = 0; tb < NBT; ++tb) x[tb] = *reinterpret_cast<const f32x4 *>(st + tb * 512 + foff);
#pragma unroll
        for (int tb = 0; tb < NBT; ++tb)
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                f32x4 q[4] = {zero, zero, zero, zero};
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    q[i / CHAIN] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[m][i], x[tb][i], q[i / CHAIN], 0, 0, 0);
                mid[m][tb] += CHAIN == 2 ? q[0] + q[1] : (q[0] + q[1]) + (q[2] + q[3]);
            }
        if ((kt & 7) == 7) {
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int tb = 0; tb < NBT; ++tb) { sum[m][tb] += mid[m][tb]; mid[m][tb] = zero; }
        }
        wr = cur;
        cur = cur + 1 == S ? 0 : cur + 1;
    }
    // the last loads (repeats of the last k-step) have to be through before their slots are written again, and
    // before the workgroup ends
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" : : : "memory");
#undef BM_F32_LOAD
    f32x4 *other = reinterpret_cast<f32x4 *>(smem) + wn * (2 * NBT * 64) + lane;
    if (ks == 1) {
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int tb = 0; tb < NBT; ++tb) other[(m * NBT + tb) * 64] = sum[m][tb] + mid[m][tb];
    }
    __syncthreads();
    if (ks == 1) return;

    // D: lane holds column r16 (activation row) and rows 4 * quad .. + 3 (weight rows)
#pragma unroll
    for (int tb = 0; tb < NBT; ++tb) {
        f32x4 v[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) v[m] = (sum[m][tb] + mid[m][tb]) + other[(m * NBT + tb) * 64];
        const int pos = row0 + tb * 16 + r16;
        if (pos >= row_end) continue;
        if (DUAL) {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[0][i] = silu_precise(v[0][i]) * v[1][i];
        }
#pragma unroll
        for (int m = 0; m < (DUAL ? 1 : 2); ++m) {
            const int n = n0 + m * 32 + wn * 16 + 4 * quad;
            float *c = static_cast<float *>(p.c) + (size_t)pos * N + n;
            if ((N & 3) == 0) {
                if (n < N) *(BM_GLOBAL f32x4 *)c = v[m];
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) if (n + i < N) c[i] = v[m][i];
            }
        }
    }
}

// The row-tile table lists each live group once, largest first (groups with more rows take longer per tile: the
// short ones fill the end of the launch).  A unit is a group and a block of output columns; up to F32_CHUNKS of its
// row tiles run side by side.  The grid holds the units of the last row tile first and those of the first one last.
// Only the first max_rows / (64 c) groups can have a row tile c, so there are few workgroups without work, and those
// do not alternate with the others: workgroups are dealt out in turn to the parts of an XCD, and a launch whose
// every second workgroup was empty ran on half of the chip (gate/up 201 -> 175 us, down 122 -> 89 us).  A unit's row
// tiles all go to one XCD, whose L2 then holds the weight block.
__host__ __device__ __forceinline__ int f32_units(int chunk, int groups, int max_rows, int n_nt) {
    const int most = chunk == 0 ? groups : max_rows / (F32_ROWS * chunk);
    return ((most < groups ? most : groups) * n_nt + 7) / 8 * 8;
}

template <bool DUAL, int CHAIN>
__global__ void __launch_bounds__(256, 3) grouped_gemm_f32_kernel(GemmParams p, int chunks, int groups, int max_rows) {
    __shared__ __attribute__((aligned(1024))) float smem[F32_STAGES * (F32_ROWS + 64) * 32];
    constexpr int BLK = DUAL ? 32 : 64;
    const int n_nt = (p.N + BLK - 1) / BLK;
    int unit = blockIdx.x, chunk = chunks - 1;
    for (; chunk > 0; --chunk) {
        const int n = f32_units(chunk, groups, max_rows, n_nt);
        if (unit < n) break;
        unit -= n;
    }
    if (unit >= p.n_mtiles[0] * n_nt) return;
    const int mt = unit / n_nt, nt = unit - mt * n_nt;
    const int g = p.mt_group[mt];
    const int end = p.offsets[g + 1];
    const size_t gofs = (size_t)(g < p.E ? g : g - p.E) * p.N * p.Kd;
    const float *b0 = static_cast<const float *>(g < p.E ? p.b0 : p.sb0) + gofs;
    const float *b1 = DUAL ? static_cast<const float *>(g < p.E ? p.b1 : p.sb1) + gofs : b0;
    // (by expert and output columns, not by the unit's number: a token's bits then do not depend on the rest of the batch)
    const int rot = (((g * ((n_nt + 7) >> 3) + (nt >> 3)) * 5) & 31) * (p.Kd >> 5) >> 5;
    const bool once = p.n_mtiles[0] > p.cached_groups && end - p.offsets[g] <= F32_ROWS;
    for (int row0 = p.offsets[g] + chunk * F32_ROWS; row0 < end; row0 += chunks * F32_ROWS) {
        const int row_end = min(end, row0 + F32_ROWS), n_rows = row_end - row0;
#define BM_F32_TILE(NBT_)                                                                                             \
    if (once) f32_tile<DUAL, NBT_, CHAIN, 2>(p, smem, b0, b1, row0, row_end, nt * BLK, rot);                                \
    else f32_tile<DUAL, NBT_, CHAIN, 0>(p, smem, b0, b1, row0, row_end, nt * BLK, rot)
        if (n_rows <= 16) { BM_F32_TILE(1); }
        else if (n_rows <= 32) { BM_F32_TILE(2); }
        else { BM_F32_TILE(4); }
#undef BM_F32_TILE
        __syncthreads();                               // the next tile's loads go where the halves met
    }
}

// The tiles load whole 128-byte lines of every row in 16-byte pieces; other reduction widths, and arrays that do not
// start on a 16-byte boundary, keep the row-by-row kernel.
template <bool DUAL>
static int launch_f32(const GemmParams &p, int max_rows, int T, hipStream_t st) {
    if (max_rows <= 0) return 0;
    if (p.Kd % 32 == 0 && aligned16(p.a) && aligned16(p.b0) && aligned16(p.b1) && aligned16(p.sb0) && aligned16(p.sb1)) {
        constexpr int BLK = DUAL ? 32 : 64;
        const int tiles = (T + F32_ROWS - 1) / F32_ROWS;          // a group rarely holds a token twice
        const int chunks = tiles < F32_CHUNKS ? tiles : F32_CHUNKS;
        const int groups = p.n_groups < max_rows ? p.n_groups : max_rows;
        const int n_nt = (p.N + BLK - 1) / BLK;
        int grid = 0;
        for (int c = 0; c < chunks; ++c) grid += f32_units(c, groups, max_rows, n_nt);
        if (p.Kd < 1024) hipLaunchKernelGGL((grouped_gemm_f32_kernel<DUAL, 1>), dim3(grid), dim3(256), 0, st, p, chunks, groups, max_rows);
        else hipLaunchKernelGGL((grouped_gemm_f32_kernel<DUAL, 2>), dim3(grid), dim3(256), 0, st, p, chunks, groups, max_rows);
    } else {
        hipLaunchKernelGGL(rowwise_f32_kernel<DUAL>, dim3(max_rows), dim3(256), (size_t)p.Kd * sizeof(float), st, p);
    }
    return launch_status(__func__);
}

int launch_gateup_f32(const GemmParams &p, int max_rows, int T, hipStream_t st) { return launch_f32<true>(p, max_rows, T, st); }
int launch_down_f32(const GemmParams &p, int max_rows, int T, hipStream_t st) { return launch_f32<false>(p, max_rows, T, st); }

}  // namespace bm
