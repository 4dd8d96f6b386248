// Grouped bf16 projections on MFMA for gfx950 (prefill-sized groups).
//
// Rows are the surviving assignments, grouped by expert; a row-tile table
// built on the device says which group each tile of BM rows belongs to.  One
// workgroup computes BM rows x 256 weight rows with fp32 accumulators (v_mfma_f32_16x16x32_bf16 in the
// main kernel - per flop it draws less power than the 32 x 32 x 16 form, and these kernels run against
// the chip's power limit - v_mfma_f32_32x32x16_bf16 in the fallbacks):
//   DUAL  : the 256 weight rows are 128 rows of W_gate and the same 128 rows
//           of W_up; the epilogue writes h = silu(g) * u as bf16.
//   !DUAL : 256 rows of W_down; the epilogue writes the product as bf16.
// Both operands have the reduction dimension contiguous, so a lane's MFMA
// operand (8 consecutive k) is one 16-byte piece of a row.
//
// Kernels, in the order the launchers prefer them:
//   grouped_gemm_mixed_k64w      persistent, k-steps of 64 with whole-line direct-to-LDS loads,
//                                v_mfma_f32_16x16x32_bf16; 256-row tiles plus one 128-row tile for a group's
//                                rest of at most 128 rows, both heights in one launch; the down projection of
//                                long reductions cuts what does not fill a round along the reduction
//   grouped_gemm256_dma          BM = 256, k-steps of 32 (reduction not a multiple of 64, offsets beyond
//                                32 bits, or a device that is not the full part)
//   grouped_gemm_bf16_kernel     BM = 128, 4 waves, register-staged double buffer, for groups too small
//                                for 256-row tiles on those shapes
// LDS rows of 128 bytes: the 64 banks span two rows, so piece p of row r is stored at slot
// p ^ ((r >> 1) & 7); the 16 lanes of one ds_read_b128 pass (16 rows, same p) then hit 16 distinct
// 16-byte slots (measured: zero bank-conflict cycles).
#include "bm_kernels.h"
#include "bm_device_shape.h"
#include "bm_tile_schedule.h"

namespace bm {

constexpr int G_BN = 256, G_BK = 64;

__device__ __forceinline__ int lds_slot(int row, int piece) { return row * G_BK + ((piece ^ ((row >> 1) & 7)) << 3); }

template <bool DUAL, int BM>
__global__ void __launch_bounds__(256) grouped_gemm_bf16_kernel(GemmParams p) {
    constexpr int THREADS = 256;                    // 4 waves, 2 x 2
    constexpr int WN = 2;                           // waves along the weight rows (2 along the rows)
    constexpr int AI = BM / 2 / 32;                 // 32-row blocks per wave
    constexpr int BJ = G_BN / WN / 32;              // 32-column blocks per wave
    constexpr int RSTEP = THREADS / 8;              // tile rows covered by one round of 16-byte loads
    constexpr int NA = BM / RSTEP, NB = G_BN / RSTEP;
    __shared__ __attribute__((aligned(16))) uint16_t sA[2][BM * G_BK];
    __shared__ __attribute__((aligned(16))) uint16_t sB[2][G_BN * G_BK];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    const int r32 = lane & 31, half = lane >> 5;

    // tile scheduling: consecutive logical tiles stay on one XCD (workgroups
    // are dealt round-robin to the 8 XCDs); see tile_of for the order inside
    const int n_mt = p.n_mtiles[0];
    const int n_nt = DUAL ? (p.N + 127) / 128 : (p.N + 255) / 256;
    const int total = n_mt * n_nt;
    const int per_xcd = (total + 7) >> 3;
    const int lid = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per_xcd || lid >= total) return;
    int mt, nt;
    tile_of(lid, n_mt, n_nt, mt, nt);

    const int g = p.mt_group[mt];
    const int row0 = p.mt_row0[mt];
    const int row_end = p.offsets[g + 1];
    const int n0 = nt * (DUAL ? 128 : 256);
    const int N = p.N, Kd = p.Kd;

    const uint16_t *a = static_cast<const uint16_t *>(p.a);
    const uint16_t *b0, *b1;
    if (g < p.E) {
        b0 = static_cast<const uint16_t *>(p.b0) + (size_t)g * N * Kd;
        b1 = DUAL ? static_cast<const uint16_t *>(p.b1) + (size_t)g * N * Kd : nullptr;
    } else {
        b0 = static_cast<const uint16_t *>(p.sb0) + (size_t)(g - p.E) * N * Kd;
        b1 = DUAL ? static_cast<const uint16_t *>(p.sb1) + (size_t)(g - p.E) * N * Kd : nullptr;
    }

    // per-thread global sources and LDS destinations
    const int lrow = tid >> 3, chunk = tid & 7;
    const uint16_t *pa[NA];
    const uint16_t *pb[NB];
    int sa_off[NA], sb_off[NB];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int r = lrow + RSTEP * i;
        const int pos = min(row0 + r, row_end - 1);
        const int src = p.row_map ? p.row_map[pos] : pos;
        pa[i] = a + (size_t)src * Kd + chunk * 8;
        sa_off[i] = lds_slot(r, chunk);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int rb = lrow + RSTEP * i;
        if (DUAL) {
            const int f = min(n0 + (rb & 127), N - 1);
            pb[i] = ((rb >> 7) ? b1 : b0) + (size_t)f * Kd + chunk * 8;
        } else {
            const int n = min(n0 + rb, N - 1);
            pb[i] = b0 + (size_t)n * Kd + chunk * 8;
        }
        sb_off[i] = lds_slot(rb, chunk);
    }

    f32x16 acc[AI][BJ];
#pragma unroll
    for (int i = 0; i < AI; ++i)
#pragma unroll
        for (int j = 0; j < BJ; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    // operand rows of this wave inside the tile
    int a_row[AI], b_row[BJ];
#pragma unroll
    for (int i = 0; i < AI; ++i) a_row[i] = wm * (BM / 2) + i * 32 + r32;
#pragma unroll
    for (int j = 0; j < BJ; ++j)
        b_row[j] = DUAL ? ((j / (BJ / 2)) * 128 + wn * (128 / WN) + (j % (BJ / 2)) * 32 + r32)
                        : (wn * (G_BN / WN) + j * 32 + r32);

    const int KT = (Kd + G_BK - 1) / G_BK;
    u32x4 ra[NA], rb[NB];
    const u32x4 zero4 = {0u, 0u, 0u, 0u};

#define BM_LOAD_GLOBAL(kt_)                                                                        \
    {                                                                                              \
        const int k0_ = (kt_) * G_BK;                                                              \
        const bool in_ = (k0_ + chunk * 8) < Kd;                                                   \
        _Pragma("unroll") for (int i = 0; i < NA; ++i) ra[i] = in_ ? ldg128(pa[i] + k0_) : zero4;  \
        _Pragma("unroll") for (int i = 0; i < NB; ++i) rb[i] = in_ ? ldg128(pb[i] + k0_) : zero4;  \
    }
#define BM_STORE_LDS(buf_)                                                                         \
    {                                                                                              \
        _Pragma("unroll") for (int i = 0; i < NA; ++i)                                             \
            *reinterpret_cast<u32x4 *>(&sA[buf_][sa_off[i]]) = ra[i];                              \
        _Pragma("unroll") for (int i = 0; i < NB; ++i)                                             \
            *reinterpret_cast<u32x4 *>(&sB[buf_][sb_off[i]]) = rb[i];                              \
    }

    BM_LOAD_GLOBAL(0);
    BM_STORE_LDS(0);
    __syncthreads();

    for (int kt = 0; kt < KT; ++kt) {
        const int buf = kt & 1;
        if (kt + 1 < KT) BM_LOAD_GLOBAL(kt + 1);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            const int piece = kk * 2 + half;
            bf16x8 fa[AI], fb[BJ];
#pragma unroll
            for (int i = 0; i < AI; ++i)
                fa[i] = as_bf16x8(*reinterpret_cast<const u32x4 *>(&sA[buf][lds_slot(a_row[i], piece)]));
#pragma unroll
            for (int j = 0; j < BJ; ++j)
                fb[j] = as_bf16x8(*reinterpret_cast<const u32x4 *>(&sB[buf][lds_slot(b_row[j], piece)]));
#pragma unroll
            for (int i = 0; i < AI; ++i)
#pragma unroll
                for (int j = 0; j < BJ; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
        }
        if (kt + 1 < KT) BM_STORE_LDS(buf ^ 1);
        __syncthreads();
    }
#undef BM_LOAD_GLOBAL
#undef BM_STORE_LDS

    // epilogue.  D[i][j]: lane holds column j = l % 32, rows 8*(v/4) + 4*(l/32) + v%4
    uint16_t *c = static_cast<uint16_t *>(p.c);
#pragma unroll
    for (int i = 0; i < AI; ++i) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = row0 + wm * (BM / 2) + i * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
            if (row >= row_end) continue;
            if (DUAL) {
#pragma unroll
                for (int jj = 0; jj < BJ / 2; ++jj) {
                    const int f = n0 + wn * (128 / WN) + jj * 32 + r32;
                    if (f < N)
                        stg16(&c[(size_t)row * N + f], f32_to_bf16(silu(acc[i][jj][v]) * acc[i][BJ / 2 + jj][v]));
                }
            } else {
#pragma unroll
                for (int j = 0; j < BJ; ++j) {
                    const int n = n0 + wn * (G_BN / WN) + j * 32 + r32;
                    if (n < N) stg16(&c[(size_t)row * N + n], f32_to_bf16(acc[i][j][v]));
                }
            }
        }
    }
}

// 256-row tiles with k-steps of 32: LDS rows are 64 bytes (4 pieces); the 64 banks span 4 rows, so piece p
// of row r sits at slot p ^ ((r >> 2) & 3).
constexpr int L_BK = 32, L_BM = 256, L_STAGE = (L_BM + G_BN) * L_BK;   // bf16 elements per stage

__device__ __forceinline__ int lds_slot32(int row, int piece) { return row * L_BK + ((piece ^ ((row >> 2) & 3)) << 3); }

// ---------------------------------------------------------------------------
// Fallback for reductions that are a multiple of 32 but not of 64.  256 rows x 256 weight rows per
// workgroup, 4 waves (2 x 2) with wave tiles of 128 x 128; the tiles go from global memory straight into
// LDS (global_load_lds_dwordx4: each lane's 16 bytes land at M0 + 16 * lane, so
// one instruction fills 16 tile rows of 64 bytes; the swizzle is applied by
// choosing which piece a lane fetches).  No staging registers, no LDS-write
// instructions, and a 5-stage ring over the whole 160 KB of LDS: the loads of
// tile kt+4 are issued in iteration kt and first needed three iterations later.
// Its 64-byte row pieces use half of every cache line they fetch, which is what
// the k-step-64 kernels below avoid.
//   iteration kt:  wait until tile kt+1 has landed (at most the 16 loads of tiles
//   kt+2, kt+3 outstanding) -> barrier (every wave's part of tile kt+1 is in LDS
//   and every wave is done with stage (kt-1)%5) -> issue tile kt+4 into stage
//   (kt+4)%5 -> MFMAs on stage kt%5, reading the first fragments of tile kt+1
//   under the last MFMAs.
// The compiler does not order LDS reads after these loads by itself, so the
// waits are explicit s_waitcnt vmcnt(n) and the barrier is a bare s_barrier.
// Needs Kd divisible by 32.
// ---------------------------------------------------------------------------
#define BM_LDS __attribute__((address_space(3)))
// s_waitcnt with only vmcnt set (gfx9 encoding: vmcnt[3:0] | expcnt 7 << 4 | lgkmcnt 15 << 8 | vmcnt[5:4] << 14)
#define BM_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 15) | (7 << 4) | (15 << 8) | (((n) >> 4) << 14))
#define BM_BARE_BARRIER() asm volatile("s_barrier" ::: "memory")

template <bool DUAL>
__global__ void __launch_bounds__(256) grouped_gemm256_dma_bf16_kernel(GemmParams p) {
    __shared__ __attribute__((aligned(1024))) uint16_t smem[5 * L_STAGE];        // 160 KB: the whole LDS
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int r32 = lane & 31, half = lane >> 5;

    const int n_mt = p.n_mtiles[0];
    const int n_nt = DUAL ? (p.N + 127) / 128 : (p.N + 255) / 256;
    const int total = n_mt * n_nt;
    const int per_xcd = (total + 7) >> 3;
    const int lid = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per_xcd || lid >= total) return;
    int mt, nt;
    tile_of(lid, n_mt, n_nt, mt, nt);

    const int g = p.mt_group[mt];
    const int row0 = p.mt_row0[mt];
    const int row_end = p.offsets[g + 1];
    const int n0 = nt * (DUAL ? 128 : 256);
    const int N = p.N, Kd = p.Kd;

    const uint16_t *a = static_cast<const uint16_t *>(p.a);
    const uint16_t *b0, *b1;
    if (g < p.E) {
        b0 = static_cast<const uint16_t *>(p.b0) + (size_t)g * N * Kd;
        b1 = DUAL ? static_cast<const uint16_t *>(p.b1) + (size_t)g * N * Kd : nullptr;
    } else {
        b0 = static_cast<const uint16_t *>(p.sb0) + (size_t)(g - p.E) * N * Kd;
        b1 = DUAL ? static_cast<const uint16_t *>(p.sb1) + (size_t)(g - p.E) * N * Kd : nullptr;
    }

    // Load instruction j of this wave fills the 1 KB block (4*j + wave) of a stage: blocks 0..15 are
    // the A tile (16 rows each), 16..31 the B tile.  Lane i supplies row 16*block + i/4, LDS slot i%4,
    // i.e. global piece (i%4) ^ ((row >> 2) & 3) = (i & 3) ^ ((i >> 4) & 3).
    const int piece = (lane & 3) ^ ((lane >> 4) & 3);
    const uint16_t *ps[8];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int r = 16 * (4 * j + wave) + (lane >> 2);         // row inside the 256-row tile
        const int pos = min(row0 + r, row_end - 1);
        const int src = p.row_map ? p.row_map[pos] : pos;
        ps[j] = a + (size_t)src * Kd + piece * 8;
        if (DUAL) {
            const int f = min(n0 + (r & 127), N - 1);
            ps[4 + j] = ((r >> 7) ? b1 : b0) + (size_t)f * Kd + piece * 8;
        } else {
            const int n = min(n0 + r, N - 1);
            ps[4 + j] = b0 + (size_t)n * Kd + piece * 8;
        }
    }

    int fa_off[2][4], fb_off[2][4];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int ar = wm * 128 + i * 32 + r32;
            const int br = DUAL ? ((i >> 1) * 128 + wn * 64 + (i & 1) * 32 + r32) : (wn * 128 + i * 32 + r32);
            fa_off[kk][i] = lds_slot32(ar, kk * 2 + half);
            fb_off[kk][i] = L_BM * L_BK + lds_slot32(br, kk * 2 + half);
        }

    f32x16 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    const int KT = Kd / L_BK;
    bf16x8 f0a[4], f0b[4], f1a[4], f1b[4];

// tile_ -> stage_: 8 direct-to-LDS loads per wave
#define BM_DMA(stage_, tile_)                                                                      \
    {                                                                                              \
        const int k0_ = min((tile_), KT - 1) * L_BK;                                               \
        uint16_t *st_ = smem + (stage_) * L_STAGE + wave * 512;                                    \
        _Pragma("unroll") for (int j = 0; j < 8; ++j)                                              \
            __builtin_amdgcn_global_load_lds((const BM_GLOBAL void *)(ps[j] + k0_),                \
                                             (BM_LDS void *)(st_ + ((j >> 2) * 16 + 4 * (j & 3)) * 512), 16, 0, 0); \
    }
#define BM_FREAD(fa_, fb_, stage_, kk_)                                                    \
    {                                                                                      \
        const uint16_t *st_ = smem + (stage_) * L_STAGE;                                   \
        _Pragma("unroll") for (int i = 0; i < 4; ++i)                                      \
            fa_[i] = as_bf16x8(*reinterpret_cast<const u32x4 *>(st_ + fa_off[kk_][i]));    \
        _Pragma("unroll") for (int i = 0; i < 4; ++i)                                      \
            fb_[i] = as_bf16x8(*reinterpret_cast<const u32x4 *>(st_ + fb_off[kk_][i]));    \
    }
#define BM_MFMA16(fa_, fb_)                                                                \
    _Pragma("unroll") for (int i = 0; i < 4; ++i)                                          \
        _Pragma("unroll") for (int j = 0; j < 4; ++j)                                      \
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa_[i], fb_[j], acc[i][j], 0, 0, 0);

    // prologue: tiles 0..3 in flight, tile 0 landed, its first fragments loaded
    BM_DMA(0, 0);
    BM_DMA(1, 1);
    BM_DMA(2, 2);
    BM_DMA(3, 3);
    BM_WAIT_VMCNT(24);
    BM_BARE_BARRIER();
    BM_FREAD(f0a, f0b, 0, 0);

    int s_cur = 0, s_nxt = 1, s_wr = 4;                // stage being multiplied, the next one, the free one
    for (int kt = 0; kt < KT; ++kt) {
        BM_WAIT_VMCNT(16);                             // tile kt+1 has landed (this wave's part)
        BM_BARE_BARRIER();                             // ... and everybody's; stage s_wr is free
        BM_FREAD(f1a, f1b, s_cur, 1);
        BM_DMA(s_wr, kt + 4);
        BM_MFMA16(f0a, f0b);
        BM_FREAD(f0a, f0b, s_nxt, 0);
        BM_MFMA16(f1a, f1b);
        _Pragma("unroll") for (int q = 0; q < 8; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // MFMA
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // DS read (f1)
        }
        _Pragma("unroll") for (int q = 0; q < 8; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);   // direct-to-LDS load
        }
        _Pragma("unroll") for (int q = 0; q < 8; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // DS read (next f0)
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 8, 0);
        s_wr = s_cur;
        s_cur = s_nxt;
        s_nxt = (s_nxt == 4) ? 0 : s_nxt + 1;
    }
    BM_WAIT_VMCNT(0);                                  // no load may land in LDS after this workgroup is gone
#undef BM_DMA
#undef BM_FREAD
#undef BM_MFMA16

    uint16_t *c = static_cast<uint16_t *>(p.c);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = row0 + wm * 128 + i * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
            if (row >= row_end) continue;
            if (DUAL) {
#pragma unroll
                for (int jj = 0; jj < 2; ++jj) {
                    const int f = n0 + wn * 64 + jj * 32 + r32;
                    if (f < N) stg16(&c[(size_t)row * N + f], f32_to_bf16(silu(acc[i][jj][v]) * acc[i][2 + jj][v]));
                }
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int n = n0 + wn * 128 + j * 32 + r32;
                    if (n < N) stg16(&c[(size_t)row * N + n], f32_to_bf16(acc[i][j][v]));
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// 256 x 256 tile with k-steps of 64 and direct-to-LDS loads that fetch whole
// 128-byte lines.  The vector cache moves one 128-byte line per two cycles
// whether a load uses all of it or half, so the 64-byte row pieces of a k-step
// of 32 cost twice the cache time of the MFMAs' data and leave the matrix cores
// waiting on load issue; here one load instruction covers 8 rows x 128 bytes.
// A k-step of 64 is two parts of 32 KB (the activation rows, the weight rows)
// and LDS holds five parts as a ring, ordered B(0) A(0) B(1) A(1) B(2) ...:
//   during k-step kt the slots hold B(kt) A(kt) B(kt+1) A(kt+1) B(kt+2).
//   One barrier per k-step, before its last 16 MFMAs (every wave has read its
//   last fragments of B(kt), A(kt) by then, and B(kt+1), A(kt+1) have landed);
//   after it A(kt+2) goes into B(kt)'s slot under the last 16 MFMAs, and B(kt+3)
//   into A(kt)'s slot spread under the next k-step's first 48 (bursts of loads
//   hold up a wave's MFMAs at issue: every instruction is hand-placed and fenced).
// LDS rows are 128 bytes, piece p of row r at slot p ^ ((r >> 1) & 7) (applied
// by choosing which global piece a lane fetches): conflict-free fragment reads.
// Needs Kd divisible by 64.
// ---------------------------------------------------------------------------
constexpr int P_PART = 256 * 64;                       // bf16 elements per part
// vmcnt and lgkmcnt in one s_waitcnt
#define BM_WAIT_VM_LGKM(vm, lgkm) \
    __builtin_amdgcn_s_waitcnt(((vm) & 15) | (7 << 4) | ((lgkm) << 8) | (((vm) >> 4) << 14))

// number of 128-row tiles: none where the plain table lists every tile
__device__ __forceinline__ int small_tiles(const GemmParams &p) { return p.mixed ? p.n_mtiles_s[0] : 0; }

// table[idx] for a wave-uniform idx through the scalar cache.  Written out by hand because the compiler
// uses scalar loads only for memory it can prove unwritten since the kernel began; behind the first
// output store it reads such tables with vector loads, and waiting for one of those means waiting for
// every direct-to-LDS load issued before it.  The tables are written by an earlier launch.
__device__ __forceinline__ int scalar_load_i32(const int32_t *table, int idx) {
    int v;
    const int off = __builtin_amdgcn_readfirstlane(idx) * 4;
    // (early clobber: the result register is none of the address registers, as a replayed load would need)
    asm volatile("s_load_dword %0, %1, %2\n\ts_waitcnt lgkmcnt(0)" : "=&s"(v) : "s"(table), "s"(off) : "memory");
    return v;
}

// The two tile loops of a launch (grouped_gemm_mixed_k64w_bf16_kernel): a group's rows are cut into 256-row tiles
// (k64w_body), and a rest of at most 128 rows becomes a 128-row tile (k64s_body).  A workgroup takes its share of the
// 256-row tiles, the plain persistent order, and its share of the 128-row tiles, which are dealt out so that the
// workgroups that got one 256-row tile fewer catch up first (SmallTileDealer).  SPLIT: cut tiles are compiled in.
__shared__ __attribute__((aligned(1024))) uint16_t k64w_smem[5 * P_PART];        // 160 KB: the whole LDS

// scratch of piece c of the cut tile t of an XCD
__device__ __forceinline__ float *partial_tile(float *splitk, const XcdWork &x, int xcd, int t, int c) {
    return splitk + (size_t)xcd * (SPLIT_XCD_TILES * SPLIT_TILE_FLOATS) + x.partial_offset(t, c);
}

// A piece of a cut tile is done: the wave leaves its fp32 accumulators in scratch memory for split_fixup_kernel
// (accumulator tile by accumulator tile, 16 bytes a lane; blocks of dead rows are left out).  Read one
// accumulator tile at a time, by hand: copies of all of them in vector registers spill.
template <int RB, int CB>
__device__ __forceinline__ void store_partial(float *dst, const f32x4 (&acc)[RB][CB], int wave_row0, int row_end) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        if (wave_row0 + i * 16 >= row_end) continue;
#pragma unroll
        for (int j = 0; j < CB; ++j)
        {
            f32x4 x;
#pragma unroll
            for (int v = 0; v < 4; ++v) asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(x[v]) : "a"(acc[i][j][v]));
            *(BM_GLOBAL f32x4 *)(dst + (i * CB + j) * 256 + lane * 4) = x;
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

template <bool DUAL, bool SPLIT>
__device__ __forceinline__ void k64w_body(const GemmParams &p, const XcdWork &work) {
    uint16_t *const smem = k64w_smem;
    constexpr int MI = 8;                                  // 16-row blocks per wave
    constexpr int NM = MI * 8;                             // MFMAs per k slice of 32
    constexpr int NR = MI + 8;                             // fragment reads per k slice
    const int tid = threadIdx.x, lane = tid & 63;
    // the wave index as a scalar: everything derived from it (LDS targets of the loads, tile halves) then
    // stays in scalar registers and costs no vector instructions in the main loop
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int r16 = lane & 15, quad = lane >> 4;           // MFMA 16x16x32: row (or column) and k eighth

    // Persistent: workgroup b serves the XCD it was dealt to (b % 8) and walks that XCD's share of the
    // logical tiles with stride XCD_WGS, so the workgroups that run together on an XCD work
    // on consecutive logical tiles (see tile_of) and a workgroup keeps its compute unit: the next tile's
    // first loads fly while the finished tile is written out, and nothing is relaunched.
    const int n_mt = p.n_mtiles[0];
    const int n_nt = DUAL ? (p.N + 127) / 128 : (p.N + 255) / 256;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int N = p.N, Kd = p.Kd;
    const int KT = Kd / 64;
    // Gate/up: the reduction is walked as a circle that each XCD enters elsewhere (see k64s_body); inside an XCD the
    // workgroups stay in step, because they share panels.  The down projection of few column tiles shares panels between
    // XCDs as well (Mixtral-shaped, 1024 tokens: 336 us in step, 345 not).
    const int rot = DUAL ? xcd * KT >> 3 : 0;
    auto rotated = [&](int k) { const int r = k + rot; return r >= KT ? r - KT : r; };
    const int R = work.nb - work.full;                 // tiles that are cut
    const int n_items = work.full + R * work.S;
    int idx = slot;                                    // next item of this workgroup
    int kbeg = 0, kend = KT;                           // k-steps of the item whose loads are being issued
    int item_tile = 0;
// next work item of this workgroup -> item_tile, kbeg, kend; false when there is none
#define BM_NEXT_ITEM(ok_)                                                                          \
    {                                                                                              \
        ok_ = idx < n_items;                                                                       \
        item_tile = idx; kbeg = 0; kend = KT;                                                      \
        if (SPLIT && ok_ && idx >= work.full && work.S > 1) {                                      \
            const int c_ = work.big_piece(idx);                                                    \
            item_tile = idx - c_ * R;                                                              \
            work.piece(c_, kbeg, kend);                                                            \
        }                                                                                          \
        idx += XCD_WGS;                                                                            \
    }
    bool have;
    BM_NEXT_ITEM(have);
    if (!have) return;
    const uint16_t *a = static_cast<const uint16_t *>(p.a);
    uint16_t *c = static_cast<uint16_t *>(p.c);

    // fragment offsets inside a part, per 32-wide k slice s: row (.. + r16), piece 4*s + quad
    int fa_off[2], fb_off[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int pc = ((4 * s + quad) ^ ((r16 >> 1) & 7)) << 3;
        fa_off[s] = (wm * (MI * 16) + r16) * 64 + pc;
        fb_off[s] = (DUAL ? (wn * 64 + r16) : (wn * 128 + r16)) * 64 + pc;
    }

    f32x4 acc[MI][8];                                  // 16 x 16 tiles: rows i*16.., columns j*16..
    bf16x8 f0a[MI], f0b[8], f1a[MI], f1b[8];
    // Load addresses are (uniform base + k offset) + a 32-bit byte offset per lane, so that the k advance
    // is scalar arithmetic and a load needs no vector address computation.
    uint32_t oa[8], ob[8];
    const uint16_t *base_b0, *base_b1;
    int row0, row_end, n0;                             // of the tile whose loads are being issued
    int g_n, row0_n, row_end_n, n0_n;                  // of the tile looked up last (BM_LOOKUP)
                                                       // (the source rows of its activation loads: in v255)
    bool n_more = false;                               // the item the loads move on to next, found a k-step
    int n_kbeg = 0, n_kend = 0;                        // before they do
    int load_tile;                                     // the tile whose loads are being issued (XCD's own number)

// Load instruction j of a wave fills the 1 KB block (4*j + wave) of a part: 8 tile rows of 128 bytes.  Lane i
// supplies row 8*block + i/8 and LDS slot i%8 of it, i.e. global piece (i % 8) ^ ((row >> 1) & 7).
// Moving the loads on to another tile takes two steps, a k-step apart:
// BM_LOOKUP(lid_): the tables of logical tile lid_ (scalar loads) and the source rows of the wave's
//   activation loads: 64 tile rows per wave, one per lane (lane l: the row load l/8 fetches for lanes
//   8 * (l%8) ..), ONE vector load of row_map.  Nothing the running loads use is touched.
// BM_ADOPT(): the load addresses of the tile looked up last; every lane picks up its eight source rows
//   from the lanes that loaded them (a lane permute; it moves data through the LDS crossbar and uses no
//   LDS memory).
// The row_map load is an assembly statement into a register the compiler does not manage (v255, named as
// clobbered so that it is allocated to the kernel; the compiler's own values stay far below it), i.e. the
// compiler neither waits for the result nor moves it.  Vector memory operations complete in issue order, so
// a wait for this load is a wait for every direct-to-LDS load issued before it; left to the compiler,
// look-up and use drained the load pipeline up to three times per tile (tile index -> group -> rows,
// dependent round trips), and given a k-step of distance it copied the pending value out of the result
// register at once and waited at the top of EVERY k-step.  By hand nothing waits at all: the look-up runs
// at the end of k-step kend - 4, BM_ADOPT at the end of k-step kend - 3, whose own wait in the middle (at
// most the 8 weight loads of its first half outstanding) has covered the row_map load.
// The lane index goes through an empty assembly statement in both: otherwise the compiler keeps the sixteen
// per-load row numbers of a lane alive across the whole tile loop, and spills them.
#define BM_LOOKUP(lid_)                                                                            \
    {                                                                                              \
        int mt_, nt_;                                                                              \
        tile_of((lid_), n_mt, n_nt, mt_, nt_);                                                     \
        g_n = scalar_load_i32(p.mt_group, mt_);                                                     \
        row0_n = scalar_load_i32(p.mt_row0, mt_);                                                   \
        row_end_n = scalar_load_i32(p.offsets, g_n + 1);                                           \
        n0_n = __builtin_amdgcn_readfirstlane(nt_) * (DUAL ? 128 : 256);                           \
        int lane_ = lane;                                                                          \
        asm volatile("" : "+v"(lane_));                                                            \
        const int r_ = 8 * (4 * (lane_ >> 3) + wave) + (lane_ & 7);                                \
        const int pos_ = min(row0_n + r_, row_end_n - 1);                                          \
        if (p.row_map)                                                                             \
            asm volatile("global_load_dword v255, %0, %1" : : "v"(pos_ * 4), "s"(p.row_map) : "v255", "memory"); \
        else                                                                                       \
            asm volatile("v_mov_b32 v255, %0" : : "v"(pos_) : "v255");                             \
    }
#define BM_ADOPT()                                                                                 \
    {                                                                                              \
        row0 = row0_n; row_end = row_end_n; n0 = n0_n;                                             \
        if (g_n < p.E) {                                                                           \
            base_b0 = static_cast<const uint16_t *>(p.b0) + (size_t)g_n * N * Kd;                  \
            base_b1 = DUAL ? static_cast<const uint16_t *>(p.b1) + (size_t)g_n * N * Kd : base_b0; \
        } else {                                                                                   \
            base_b0 = static_cast<const uint16_t *>(p.sb0) + (size_t)(g_n - p.E) * N * Kd;         \
            base_b1 = DUAL ? static_cast<const uint16_t *>(p.sb1) + (size_t)(g_n - p.E) * N * Kd : base_b0; \
        }                                                                                          \
        int lane_ = lane, rmv_;                                                                    \
        asm volatile("" : "+v"(lane_));                                                            \
        asm volatile("v_mov_b32 %0, v255" : "=v"(rmv_));                                           \
        _Pragma("unroll") for (int j = 0; j < 8; ++j) {                                            \
            const int r_ = 8 * (4 * j + wave) + (lane_ >> 3);                                      \
            const int piece_ = (lane_ & 7) ^ ((r_ >> 1) & 7);                                      \
            const int src_ = __builtin_amdgcn_ds_bpermute(4 * (8 * j + (lane_ >> 3)), rmv_);       \
            oa[j] = ((uint32_t)src_ * (uint32_t)Kd + piece_ * 8) * 2u;                             \
            /* DUAL: rows 0-127 of the part are W_gate rows (loads 0-3), rows 128-255 W_up rows (4-7) */ \
            const int n_ = DUAL ? min(n0 + (r_ & 127), N - 1) : min(n0 + r_, N - 1);               \
            ob[j] = ((uint32_t)n_ * (uint32_t)Kd + piece_ * 8) * 2u;                               \
        }                                                                                          \
    }
// load j_ of the activation part (A) / weight part (B) of k-step tile_ into slot_
#define BM_DMA_AT(base_, off_, slot_, tile_, j_)                                                   \
    __builtin_amdgcn_global_load_lds(                                                              \
        (const BM_GLOBAL void *)(reinterpret_cast<const char *>((base_) + rotated(min((tile_), kend - 1)) * 64) + (off_)), \
        (BM_LDS void *)(smem + (slot_) * P_PART + wave * 512 + (j_) * 2048), 16, 0, 0)
#define BM_DMA_A(slot_, tile_, j_) BM_DMA_AT(a, oa[j_], slot_, tile_, j_)
#define BM_DMA_B(slot_, tile_, j_) BM_DMA_AT(((j_) < 4 ? base_b0 : base_b1), ob[j_], slot_, tile_, j_)
// B(0) A(0) B(1) A(1) of the tile set up last into slots 0..3
#define BM_PROLOGUE()                                                                              \
    {                                                                                              \
        _Pragma("unroll") for (int j = 0; j < 8; ++j) BM_DMA_B(0, kbeg, j);                        \
        _Pragma("unroll") for (int j = 0; j < MI; ++j) BM_DMA_A(1, kbeg, j);                       \
        _Pragma("unroll") for (int j = 0; j < 8; ++j) BM_DMA_B(2, kbeg + 1, j);                    \
        _Pragma("unroll") for (int j = 0; j < MI; ++j) BM_DMA_A(3, kbeg + 1, j);                   \
    }
#define BM_LD(ptr_) as_bf16x8(*reinterpret_cast<const u32x4 *>(ptr_))
// weight fragment j of 8: 16 weight rows; DUAL: fragments 0-3 are W_gate rows, 4-7 the same rows of W_up
#define BM_BOFF(j_) (DUAL ? (((j_) >> 2) * 8192 + ((j_) & 3) * 1024) : (j_) * 1024)
// fragment read d_ of NR, in the order the MFMAs need them: a0 b0..b7 a1..a(MI-1)
#define BM_RD(d_, fa_, fb_, sa_, sb_)                                                              \
    {                                                                                              \
        if ((d_) == 0) fa_[0] = BM_LD(sa_);                                                        \
        else if ((d_) <= 8) fb_[(d_) - 1] = BM_LD((sb_) + BM_BOFF((d_) - 1));                      \
        else fa_[(d_) - 8] = BM_LD((sa_) + ((d_) - 8) * 1024);                                     \
    }
// The MFMA is written as an assembly statement with the accumulator tied to an AGPR tile as input and
// output.  With the builtin the register allocator lets accumulator tiles change registers across the loop
// (down projection: a loop full of copies, measured 70 % slower) and copies all 256 accumulator values to
// vector registers where the loop ends (gate/up projection: up to 48 registers spilled around the
// write-out, and every reload from scratch memory waits for all loads and stores in flight).  The
// compiler's hazard recogniser does not see inside the statement, so the two distances it would otherwise
// guarantee are put in by hand, as s_nop statements that carry a data dependency on the accumulator
// concerned (an instruction-scheduling fence in those places makes the register allocator spill about 200
// registers):
//   - accumulator zeroing (VALU writes of the AGPRs) -> first MFMA, which reads acc[0][0] as its third
//     operand: at most 2 wait states are required on this family; 8 are inserted behind the zeroing
//     (a barrier and the first 16 fragment reads follow before that MFMA can issue anyway).  The zeroing of
//     the other accumulators cannot move closer to their first MFMA than that because the k-steps of a tile
//     form ONE loop and the zeroing stays in front of it.  Do not peel the first k-step off that loop: in
//     straight-line code the compiler sinks each accumulator's zeroing to right in front of its first MFMA,
//     which then reads the stale register (every 128-row tile came out wrong when this was tried; tying a
//     wait to all 64 accumulators instead made the allocator spill 128 registers);
//   - last MFMA of a tile (acc[MI - 1][7]) -> first read of an accumulator by another instruction (write-out,
//     partial-tile store): an 8-pass MFMA result needs 11 wait states (18 for a 16-pass one); 32 are
//     inserted where the write-out starts.  Every other accumulator's MFMA is at least 16 cycles older.  The write-outs
//     read accumulators through assembly statements (volatile, so in order behind the wait): where the compiler reads them by
//     itself it also moves the accumulator that the wait is tied to, in front of the wait.
// Inside the loop an accumulator is next touched by its own MFMA 63 instructions later (same register as
// destination and third operand), which the MFMA pipeline interlocks by itself.
// Down projection: the weight fragment is the first operand, so the product comes out transposed, i.e. a
// lane holds four consecutive output columns (4 * quad ...) of one output row (r16), which pack into 8
// contiguous bytes (3-9 % faster through the shorter write-out; the gate/up projection measured 1-3 %
// slower with that order and keeps activations first).
#define BM_MFMA1(m_, fa_, fb_)                                                                     \
    {                                                                                              \
        if (DUAL)                                                                                  \
            asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0"                                          \
                : "+a"(acc[(m_) >> 3][(m_) & 7]) : "v"(fa_[(m_) >> 3]), "v"(fb_[(m_) & 7]));       \
        else                                                                                       \
            asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0"                                          \
                : "+a"(acc[(m_) >> 3][(m_) & 7]) : "v"(fb_[(m_) & 7]), "v"(fa_[(m_) >> 3]));       \
    }

    BM_LOOKUP(work.big0 + item_tile);
    load_tile = item_tile;
    BM_WAIT_VM_LGKM(0, 0);                             // the row_map load, which the compiler does not wait for
    BM_ADOPT();
    BM_PROLOGUE();
    // The ring runs on across tiles: during the last two k-steps of a tile the loads already fetch the
    // first two k-steps of the workgroup's next item (instead of repeats of the last k-step), so a new
    // tile starts with its operands in LDS and nothing is drained in between.
    int sB = 0, sA = 1, sAp = 4;                       // slots of B(kt), A(kt), and of A(kt-1) (free)
    // first tile: B(0) and A(0) have landed - vector memory operations complete in issue order and only
    // the loads of B(1), A(1) are younger
    BM_WAIT_VMCNT(8 + MI);
    for (;;) {
        const int t_row0 = row0, t_row_end = row_end, t_n0 = n0;    // the tile being multiplied
        const int t_tile = load_tile;
        const int t_kbeg = kbeg, t_kend = kend;
        bool more = false;                             // the loads have moved on to a next item (uniform)
        // One tile: accumulators cleared, then the k-steps.  Written as a macro so that the down projection
        // can also instantiate it without the matrix work (COMPUTE_ = false, see below); the steps, in order:
        //  - barrier: every wave's part of B(0), A(0) is in LDS (first tile: the wait above; later tiles: they
        //    were waited for in the middle of the previous tile's last k-step), and every wave is done with the
        //    write-out staging in the slot the first loads of this tile will fill; first fragments read.
        //  - per k-step, kl = the k-step its loads fetch: two ahead, in the next item once this one is through.
        //  - first k slice of 32: 64 MFMAs; the second slice's fragments are read under MFMAs 0-31 (one read
        //    per two MFMAs), the 8 loads of B(kt+2) go into the slot A(kt-1) has left, one under every eighth
        //    MFMA (spread evenly: bunched loads hold up the MFMAs behind them at issue; measured 5 % on the
        //    whole kernel).
        //  - wait + barrier: every fragment of B(kt), A(kt) is in registers; A(kt+1), B(kt+1) have landed (this
        //    wave's part: at most the 8 loads of B(kt+2) are outstanding - whatever was issued before them, the
        //    previous tile's stores included, is complete); after the barrier both hold for every wave.
        //  - second slice: A(kt+2) goes into the slot B(kt) has left, one load under every eighth MFMA; the
        //    first fragments of k-step kt+1 are read under the first half, so that none of them is still in
        //    flight when the next k-step starts (after the last k-step of a tile they are the next tile's and
        //    are read again at its start: no register stays live across the write-out).
        //  - three k-steps before the end the loads of this item are all issued: from here on they fetch the
        //    next one, which was looked up a k-step earlier (BM_LOOKUP, BM_ADOPT).
#define BM_TILE_LOOP(COMPUTE_)                                                                                        \
    {                                                                                                                 \
        if (COMPUTE_) {                                                                                               \
            _Pragma("unroll") for (int i = 0; i < MI; ++i)                                                            \
                _Pragma("unroll") for (int j = 0; j < 8; ++j)                                                         \
                    _Pragma("unroll") for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.0f;                                \
            asm volatile("s_nop 7" : "+a"(acc[0][0]));  /* acc[0][0]: the first MFMA's accumulator */       \
        }                                                                                                             \
        BM_BARE_BARRIER();                                                                                            \
        {                                                                                                             \
            const uint16_t *sa_ = smem + sA * P_PART + fa_off[0];                                                     \
            const uint16_t *sb_ = smem + sB * P_PART + fb_off[0];                                                     \
        _Pragma("unroll")                                                                                             \
            for (int d = 0; (COMPUTE_) && d < NR; ++d) BM_RD(d, f0a, f0b, sa_, sb_)                                   \
        }                                                                                                             \
        for (int kt = t_kbeg; kt < t_kend; ++kt) {                                                                    \
            const int kl = more ? kbeg + (kt + 2 - t_kend) : kt + 2;                                                  \
            /* no LDS read is pending here (the last ones were issued half a k-step ago); said explicitly,  */        \
            /* because the compiler otherwise puts its own wait for the loop-carried fragments behind this */        \
            /* k-step's first read and the first MFMA stalls for an LDS round trip */                                 \
            BM_WAIT_VM_LGKM(63, 0);                                                                                   \
            {                                                                                                         \
                const uint16_t *sa_ = smem + sA * P_PART + fa_off[1];                                                 \
                const uint16_t *sb_ = smem + sB * P_PART + fb_off[1];                                                 \
        _Pragma("unroll")                                                                                             \
                for (int m = 0; m < NM; ++m) {                                                                        \
                    if (COMPUTE_) BM_MFMA1(m, f0a, f0b);                                                              \
                    if ((COMPUTE_) && m < 2 * NR && (m & 1) == 0) BM_RD(m >> 1, f1a, f1b, sa_, sb_)                   \
                    if ((m & 7) == 5) BM_DMA_B(sAp, kl, m >> 3);                                                      \
                    __builtin_amdgcn_sched_barrier(0);                                                                \
                }                                                                                                     \
            }                                                                                                         \
            BM_WAIT_VM_LGKM(8, 0);                                                                                    \
            BM_BARE_BARRIER();                                                                                        \
            const int sBn = sB >= 3 ? sB - 3 : sB + 2, sAn = sA >= 3 ? sA - 3 : sA + 2;                               \
            {                                                                                                         \
                const uint16_t *sa_ = smem + sAn * P_PART + fa_off[0];                                                \
                const uint16_t *sb_ = smem + sBn * P_PART + fb_off[0];                                                \
        _Pragma("unroll")                                                                                             \
                for (int m = 0; m < NM; ++m) {                                                                        \
                    if (COMPUTE_) BM_MFMA1(m, f1a, f1b);                                                              \
                    if ((m & 7) == 1) BM_DMA_A(sB, kl, m >> 3);                                                       \
                    if ((COMPUTE_) && m < 2 * NR && (m & 1) == 0) BM_RD(m >> 1, f0a, f0b, sa_, sb_)                   \
                    __builtin_amdgcn_sched_barrier(0);                                                                \
                }                                                                                                     \
            }                                                                                                         \
            sAp = sA;                                                                                                 \
            sB = sBn;                                                                                                 \
            sA = sAn;                                                                                                 \
            if (kt == t_kend - 3) {                                                                                   \
                more = n_more;                                                                                        \
                if (more) {                                                                                           \
                    kbeg = n_kbeg; kend = n_kend; load_tile = item_tile;                                               \
                    BM_ADOPT();                                                                                       \
                }                                                                                                     \
            } else if (kt == t_kend - 4) {    /* every item has at least 4 k-steps */                                  \
                const int kb_ = kbeg, ke_ = kend;                                                                     \
                BM_NEXT_ITEM(n_more);                                                                                 \
                n_kbeg = kbeg; n_kend = kend;                                                                         \
                kbeg = kb_; kend = ke_;                                                                               \
                if (n_more) BM_LOOKUP(work.big0 + item_tile);                                                         \
            }                                                                                                         \
        }                                                                                                             \
    }
        // Down projection of 256-row tiles alone (SPLIT; a launch of both heights has no such tile): a tile of at most
        // 128 rows leaves the two waves of the lower row half nothing but padding.  They keep their share of the loads, the waits and the barriers - the same instruction
        // stream minus every MFMA and fragment read - and skip the write-out: the chip runs these kernels
        // against its power limit, and what the idle matrix cores do not draw lets the others clock higher
        // (Qwen3-shaped layer, 41 % padding: down projection -6 %).
        const bool live = !SPLIT || !(wm == 1 && t_row_end - t_row0 <= MI * 16);
        if (!SPLIT || live) BM_TILE_LOOP(true)
        else BM_TILE_LOOP(false)
#undef BM_TILE_LOOP
        // The tile is done.  The slot A(last k-step) sat in is free for every wave since the barrier in
        // the middle of that k-step; it stages the write-out while the next tile's loads land elsewhere.

        const bool t_partial = SPLIT && t_kend - t_kbeg < KT;
        if (!live && !t_partial) {                     // nothing but padding rows: nothing to write
            if (!more) break;
            continue;
        }
        // last MFMA of the tile -> first read of an accumulator (see BM_MFMA1): acc[MI - 1][7] is the last MFMA's
        // accumulator, every other one is at least one MFMA (16 cycles) older
        asm volatile("s_nop 15\n\ts_nop 15" : "+a"(acc[MI - 1][7]));
        if (t_partial) {
            if (live)
                store_partial<MI, 8>(partial_tile(p.splitk, work, xcd, t_tile - work.full, work.piece_at(t_kbeg)) + wave * (MI * 8 * 256), acc,
                                     t_row0 + wm * (MI * 16), t_row_end);
            if (!more) break;
            continue;
        }

        // Write-out through the free slot (8 KB per wave).  Gate/up: an accumulator tile holds, per lane, four
        // rows of one column; 16 rows at a time are laid out row-major in LDS as bf16 - neighbouring lanes
        // swap one value so that every lane writes a packed pair - and read back as 16-byte pieces, so a
        // store instruction writes whole 128-byte lines.  A wave uses only its own region and LDS
        // operations of a wave stay in order.
        if (DUAL) {
            // gate/up: accumulator tiles are (row 4 * quad + v, column r16) - four rows of one column per lane
            constexpr int OC = 4;                       // 16-column output blocks per wave
            constexpr int SD = 36;                      // LDS row stride in dwords (padded against conflicts)
            constexpr int PR = OC * 2;                  // 16-byte pieces per output row
            uint32_t *stage = reinterpret_cast<uint32_t *>(smem + sAp * P_PART) + wave * 2048;
            // The accumulators are read one pair of values at a time, by hand and behind scheduling fences:
            // left to itself the compiler copies all 256 of them to vector registers where the loop ends
            // and spills what does not fit, and every reload waits for all stores issued so far.  The lane
            // index is hidden from it for the same reason (its derived constants stayed live across tiles).
            int lane_w = lane;
            asm volatile("" : "+v"(lane_w));
            const int r16 = lane_w & 15, quad = lane_w >> 4;
            const bool odd = lane_w & 1;
#pragma unroll
            for (int i = 0; i < MI; ++i) {
#pragma unroll
                for (int j = 0; j < OC; ++j) {
#pragma unroll
                    for (int v = 0; v < 4; v += 2) {
                        float g0, g1, u0, u1;
                        asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(g0) : "a"(acc[i][j][v]));
                        asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(g1) : "a"(acc[i][j][v + 1]));
                        asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(u0) : "a"(acc[i][4 + j][v]));
                        asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(u1) : "a"(acc[i][4 + j][v + 1]));
                        const float x0 = silu(g0) * u0;
                        const float x1 = silu(g1) * u1;
                        // even lane keeps row v and gets the right-hand neighbour's value of that row;
                        // odd lane keeps row v+1 and gets the left-hand neighbour's
                        const float send = odd ? x0 : x1;
                        const float recv = __builtin_bit_cast(
                            float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, send), 0xB1, 0xF, 0xF, true));
                        const uint32_t pk = odd ? pack_bf16x2(recv, x1) : pack_bf16x2(x0, recv);
                        const int lrow = 4 * quad + v + (odd ? 1 : 0);
                        stage[lrow * SD + j * 8 + (r16 >> 1)] = pk;
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int t = 0; t < PR / 4; ++t) {
                    const int q = lane_w + 64 * t;
                    const int lrow = q / PR, pc = q % PR;
                    const u32x4 val = *reinterpret_cast<const u32x4 *>(stage + lrow * SD + pc * 4);
                    const int row = t_row0 + wm * (MI * 16) + i * 16 + lrow;
                    const int col = t_n0 + wn * (OC * 16) + pc * 8;
                    if (row < t_row_end && col < N) stg128(&c[(size_t)row * N + col], val);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            // Down projection (weights as the first MFMA operand): an accumulator tile holds, per lane, four
            // consecutive columns of one row (row r16, columns 4 * quad ...), i.e. 8 contiguous bytes of
            // bf16: one LDS write per accumulator tile and no lane exchange.
            constexpr int OC = 8;                       // 16-column output blocks per wave
            constexpr int SD = 68;                      // LDS row stride in dwords (16-byte aligned, rows 4 banks apart)
            constexpr int PR = OC * 2;                  // 16-byte pieces per output row
            uint32_t *stage = reinterpret_cast<uint32_t *>(smem + sAp * P_PART) + wave * 2048;
#pragma unroll
            for (int i = 0; i < MI; ++i) {
#pragma unroll
                for (int j = 0; j < OC; ++j) {
                    float x[4];
#pragma unroll
                    for (int v = 0; v < 4; ++v) asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(x[v]) : "a"(acc[i][j][v]));
                    u32x2 pk;
                    pk[0] = pack_bf16x2(x[0], x[1]);
                    pk[1] = pack_bf16x2(x[2], x[3]);
                    *reinterpret_cast<u32x2 *>(stage + r16 * SD + j * 8 + 2 * quad) = pk;
                }
#pragma unroll
                for (int t = 0; t < PR / 4; ++t) {
                    const int q = lane + 64 * t;
                    const int lrow = q / PR, pc = q % PR;
                    const u32x4 val = *reinterpret_cast<const u32x4 *>(stage + lrow * SD + pc * 4);
                    const int row = t_row0 + wm * (MI * 16) + i * 16 + lrow;
                    const int col = t_n0 + wn * (OC * 16) + pc * 8;
                    if (row < t_row_end && col < N) stg128(&c[(size_t)row * N + col], val);
                }
            }
        }
        if (!more) break;
    }
    // the last tile's loads ran past its end (repeats of its last k-step): nothing may still be landing in
    // LDS when the workgroup ends
    BM_WAIT_VM_LGKM(0, 0);
#undef BM_LOOKUP
#undef BM_ADOPT
#undef BM_NEXT_ITEM
#undef BM_PROLOGUE
#undef BM_DMA_AT
#undef BM_DMA_A
#undef BM_DMA_B
#undef BM_LD
#undef BM_BOFF
#undef BM_RD
#undef BM_MFMA1
}

// ---------------------------------------------------------------------------
// 128 x 256 tile, the only user of its weight panel: bound by streaming that panel from memory.
//   Stages: a k-step is 48 KB (weight rows, then activation rows) and LDS holds three of them; the loads of
//   k-step kt + 3 go out in the second half of k-step kt, once its fragments are in registers, and are waited for
//   in the middle of k-step kt + 2: 24 loads (24 KB) a wave in flight, twice what the 256-row ring leaves them.
//   Waves: each owns 64 weight rows and all 128 activation rows, so a weight fragment is read from LDS once.
//   Streaming: the weights are loaded non-temporally (STREAM; they are not read again, and would push activations and
//   router matrix out of the L2: Qwen3-shaped layer at 512 tokens, gate/up 85 -> 79 us, the next front kernel 19.4 -> 15.6),
//   unless those of the live groups are few enough to stay in the 256 MB memory-side cache until the next call (cached_groups);
//   and the tiles of an XCD enter the reduction at 32 different places and walk it as a circle: weight rows lie a
//   multiple of 4 KB apart in many layers, and workgroups in step all ask the same memory channels (256 units reading
//   panels of 256 rows of 4 / 8 KB: 4.2 TB/s in step, 5.9 / 6.1 TB/s from 32 places, 6.5 / 6.7 non-temporally too; 1.5 KB
//   rows 4.6 -> 5.5, 28 KB rows 6.0 -> 7.0).  What an XCD misses in its L2 comes at 7 TB/s for the whole chip, from the
//   memory-side cache as well.
// Kernel times, 128-row tiles on the 256-row ring | here, us: Mixtral-shaped 256 tokens gate/up 292 | 250, Qwen3-shaped 512
// tokens 88 | 79 and 52 | 52, 2048 tokens 156 | 148, DeepSeek-shaped 128 tokens 53 | 46 and 36 | 33.
// Hazards around the assembly MFMA as in k64w_body.
// ---------------------------------------------------------------------------
constexpr int DMA_STREAM = 2;                              // cache policy of a load that is not read again (nt)

// Write-out of a 128-row tile, or of its first 16 * RBL rows: 16 rows at a time through the wave's own 4 KB of LDS (stage)
// into 16-byte stores, as in k64w_body.  wcol0: first output column of the wave.
template <bool DUAL, int RBL, int NJ>
__device__ __forceinline__ void k64s_write(const f32x4 (&acc)[RBL][NJ], uint32_t *stage, uint16_t *c, int N, int t_row0, int t_row_end, int wcol0,
                                           int t_n_end, int lane) {
    if (DUAL) {
        constexpr int OC = NJ / 2;                  // 16-column output blocks per wave
        constexpr int SD = 20;
        int lane_w = lane;
        asm volatile("" : "+v"(lane_w));
        const int r16 = lane_w & 15, quad = lane_w >> 4;
        const bool odd = lane_w & 1;
#pragma unroll
        for (int i = 0; i < RBL; ++i) {
            if (NJ == 4 && t_row0 + i * 16 >= t_row_end) break;
#pragma unroll
            for (int j = 0; j < OC; ++j) {
#pragma unroll
                for (int v = 0; v < 4; v += 2) {
                    float g0, g1, u0, u1;
                    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(g0) : "a"(acc[i][j][v]));
                    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(g1) : "a"(acc[i][j][v + 1]));
                    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(u0) : "a"(acc[i][OC + j][v]));
                    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(u1) : "a"(acc[i][OC + j][v + 1]));
                    const float x0 = silu(g0) * u0;
                    const float x1 = silu(g1) * u1;
                    const float send = odd ? x0 : x1;
                    const float recv = __builtin_bit_cast(
                        float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, send), 0xB1, 0xF, 0xF, true));
                    const uint32_t pk = odd ? pack_bf16x2(recv, x1) : pack_bf16x2(x0, recv);
                    const int lrow = 4 * quad + v + (odd ? 1 : 0);
                    stage[lrow * SD + j * 8 + (r16 >> 1)] = pk;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            const int lrow = lane_w / (2 * OC) % 16, pc = lane_w % (2 * OC);
            const u32x4 val = *reinterpret_cast<const u32x4 *>(stage + lrow * SD + pc * 4);
            const int row = t_row0 + i * 16 + lrow, col = wcol0 + pc * 8;
            if (lane_w < 32 * OC && row < t_row_end && col < t_n_end) stg128(&c[(size_t)row * N + col], val);
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
        constexpr int SD = 36;
        const int r16 = lane & 15, quad = lane >> 4;
        u32x4 val[2][NJ / 2];                       // a block's pieces are stored once the next block's are on their way
        auto store = [&](int i) {
#pragma unroll
            for (int t = 0; t < NJ / 2; ++t) {
                const int q = lane + 64 * t;
                const int row = t_row0 + i * 16 + q / (2 * NJ), col = wcol0 + q % (2 * NJ) * 8;
                if (row < t_row_end && col < t_n_end) stg128(&c[(size_t)row * N + col], val[i & 1][t]);
            }
        };
#pragma unroll
        for (int i = 0; i < RBL; ++i) {
            if (t_row0 + i * 16 < t_row_end) {
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    float x[4];
#pragma unroll
                    for (int v = 0; v < 4; ++v) asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(x[v]) : "a"(acc[i][j][v]));
                    u32x2 pk;
                    pk[0] = pack_bf16x2(x[0], x[1]);
                    pk[1] = pack_bf16x2(x[2], x[3]);
                    *reinterpret_cast<u32x2 *>(stage + r16 * SD + j * 8 + 2 * quad) = pk;
                }
#pragma unroll
                for (int t = 0; t < NJ / 2; ++t) {
                    const int q = lane + 64 * t;
                    val[i & 1][t] = *reinterpret_cast<const u32x4 *>(stage + q / (2 * NJ) * SD + q % (2 * NJ) * 4);
                }
            }
            if (i > 0) store(i - 1);
        }
        store(RBL - 1);
    }
}

template <bool DUAL, bool SPLIT, bool STREAM, int NJ>
__device__ __forceinline__ void k64s_body(const GemmParams &p, const XcdWork &work, const SmallPlan &plan) {
    constexpr int RB = 8;                                  // 16-row blocks of the tile
    uint16_t *const smem = k64w_smem;
    static_assert(NJ == 4 || NJ == 2, "16-column weight blocks per wave (DUAL: half of them of either matrix)");
    constexpr int NB = 2 * NJ;                             // weight loads per wave and k-step
    constexpr int BROWS = 64 * NJ;                         // weight rows of the tile
    constexpr int NA = RB / 2;                             // activation loads per wave and k-step
    constexpr int NL = NA + NB;                            // loads per wave and k-step
    constexpr int STAGE = (BROWS + RB * 16) * 64;           // bf16 elements of a stage: weight rows, then activation rows
    constexpr int NS = NJ == 4 ? 3 : 4;                    // stages
    static_assert(NS * STAGE + 4 * 1024 * 2 <= 5 * P_PART, "the stages leave 4 KB per wave for the write-out");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, quad = lane >> 4;
    constexpr int BLK = DUAL ? 16 : 32;                    // columns by which the width of a tile varies
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int N = p.N, Kd = p.Kd;
    const int KT = Kd / 64;
    const bool WIDE = NJ == 4 && plan.cols == (DUAL ? (N + 127) / 128 : (N + 255) / 256);   // column tiles of full width
    const int cols = plan.cols, n_blk = N / BLK, n_halves = 2 * plan.halved * cols;   // items that are halves of 256-row tiles
    int rot = 0, rot_n = 0;                                // where the tile whose loads are being issued enters the reduction
    auto rotated = [&](int k) { const int r = k + rot; return r >= KT ? r - KT : r; };
    SmallTileDealer dealer;
    dealer.init((work.nb - work.full) * work.S + work.full, work.ns * work.S, XCD_WGS, slot);
    int item = 0, kbeg = 0, kend = KT;
#define BM_NEXT_ITEM(ok_, kb_, ke_)                                                                \
    {                                                                                              \
        kb_ = 0; ke_ = KT;                                                                         \
        ok_ = dealer.next(item);                                                                   \
        if (SPLIT && ok_ && work.S > 1) {                                                          \
            const int c_ = work.small_piece(item);                                                 \
            item -= c_ * work.ns;                                                                  \
            work.piece(c_, kb_, ke_);                                                              \
        }                                                                                          \
    }
    bool n_more;
    BM_NEXT_ITEM(n_more, kbeg, kend);
    if (!n_more) return;
    const uint16_t *a = static_cast<const uint16_t *>(p.a);
    uint16_t *c = static_cast<uint16_t *>(p.c);
    int fa_off[2], fb_off[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int pc = ((4 * s + quad) ^ ((r16 >> 1) & 7)) << 3;
        fa_off[s] = BROWS * 64 + r16 * 64 + pc;
        fb_off[s] = (wave * (DUAL ? NJ * 8 : NJ * 16) + r16) * 64 + pc;
    }
    bf16x8 f0a[RB], f0b[NJ], f1a[RB], f1b[NJ];
    uint32_t oa[NA], ob[NB];
    const uint16_t *base_b0, *base_b1;
    int row0, row_end, n0, n_end;
    int g_n, row0_n, row_end_n, n0_n, n_end_n;
#define BM_LOOKUP(lid_)                                                                            \
    {                                                                                              \
        const int id_ = __builtin_amdgcn_readfirstlane(lid_);                                      \
        const bool half_ = id_ < n_halves;             /* the halves of a tile follow each other */ \
        const int q_ = half_ ? id_ >> 1 : id_ - n_halves;                                          \
        const int mt_ = q_ / cols, ct_ = q_ - mt_ * cols;                                          \
        g_n = scalar_load_i32(half_ ? p.mt_group : p.mt_group_s, mt_);                             \
        row0_n = scalar_load_i32(half_ ? p.mt_row0 : p.mt_row0_s, mt_) + (half_ ? (id_ & 1) * 128 : 0); \
        row_end_n = scalar_load_i32(p.offsets, g_n + 1);                                           \
        n0_n = WIDE ? ct_ * (DUAL ? BROWS / 2 : BROWS) : __builtin_amdgcn_readfirstlane(ct_ * n_blk / cols) * BLK; \
        n_end_n = WIDE ? min(n0_n + (DUAL ? BROWS / 2 : BROWS), N) : __builtin_amdgcn_readfirstlane((ct_ + 1) * n_blk / cols) * BLK; \
        rot_n = (((half_ ? q_ : id_ - work.small0) * 5) & 31) * KT >> 5;                           \
        int lane_ = lane;                                                                          \
        asm volatile("" : "+v"(lane_));                                                            \
        const int r_ = 8 * (4 * (lane_ >> 3) + wave) + (lane_ & 7);                                \
        const int pos_ = min(row0_n + r_, row_end_n - 1);                                          \
        if (p.row_map)                                                                             \
            asm volatile("global_load_dword v255, %0, %1" : : "v"(pos_ * 4), "s"(p.row_map) : "v255", "memory"); \
        else                                                                                       \
            asm volatile("v_mov_b32 v255, %0" : : "v"(pos_) : "v255");                             \
    }
#define BM_ADOPT()                                                                                 \
    {                                                                                              \
        row0 = row0_n; row_end = row_end_n; n0 = n0_n; n_end = n_end_n; rot = rot_n;               \
        if (g_n < p.E) {                                                                           \
            base_b0 = static_cast<const uint16_t *>(p.b0) + (size_t)g_n * N * Kd;                  \
            base_b1 = DUAL ? static_cast<const uint16_t *>(p.b1) + (size_t)g_n * N * Kd : base_b0; \
        } else {                                                                                   \
            base_b0 = static_cast<const uint16_t *>(p.sb0) + (size_t)(g_n - p.E) * N * Kd;         \
            base_b1 = DUAL ? static_cast<const uint16_t *>(p.sb1) + (size_t)(g_n - p.E) * N * Kd : base_b0; \
        }                                                                                          \
        int lane_ = lane, rmv_;                                                                    \
        asm volatile("" : "+v"(lane_));                                                            \
        asm volatile("v_mov_b32 %0, v255" : "=v"(rmv_));                                           \
        _Pragma("unroll") for (int j = 0; j < (NA > NB ? NA : NB); ++j) {                                          \
            const int r_ = 8 * (4 * j + wave) + (lane_ >> 3);                                      \
            const int piece_ = (lane_ & 7) ^ ((r_ >> 1) & 7);                                      \
            if (j < NA) {                                                                          \
                const int src_ = __builtin_amdgcn_ds_bpermute(4 * (8 * j + (lane_ >> 3)), rmv_);   \
                oa[j] = ((uint32_t)src_ * (uint32_t)Kd + piece_ * 8) * 2u;                         \
            }                                                                                      \
            if (j < NB) {                                                                          \
                const int n_ = min(n0 + (DUAL ? r_ % (BROWS / 2) : r_), n_end - 1);                \
                ob[j] = ((uint32_t)n_ * (uint32_t)Kd + piece_ * 8) * 2u;                           \
            }                                                                                      \
        }                                                                                          \
    }
#define BM_DMA_AT(base_, off_, dst_, tile_, aux_)                                                  \
    __builtin_amdgcn_global_load_lds(                                                              \
        (const BM_GLOBAL void *)(reinterpret_cast<const char *>((base_) + rotated(min((tile_), kend - 1)) * 64) + (off_)), \
        (BM_LDS void *)(smem + (dst_) + wave * 512), 16, 0, aux_)
// load j_ of NL of k-step tile_ into stage st_: the weight rows first
#define BM_DMA(st_, tile_, j_)                                                                     \
    {                                                                                              \
        if ((j_) < NB) BM_DMA_AT(((j_) < NJ ? base_b0 : base_b1), ob[(j_) % NB], (st_) * STAGE + (j_) * 2048, tile_, STREAM ? DMA_STREAM : 0); \
        else BM_DMA_AT(a, oa[((j_) - NB) % NA], (st_) * STAGE + BROWS * 64 + ((j_) - NB) * 2048, tile_, 0); \
    }
#define BM_LD(ptr_) as_bf16x8(*reinterpret_cast<const u32x4 *>(ptr_))
#define BM_BOFF(j_) (DUAL ? ((j_) / (NJ / 2) * (BROWS * 32) + (j_) % (NJ / 2) * 1024) : (j_) * 1024)
// fragment read d_ of NR, in the order the MFMAs need them: a0 b0..b3 a1..
#define BM_RD(d_, fa_, fb_, st_, s_)                                                               \
    {                                                                                              \
        const uint16_t *sp_ = smem + (st_) * STAGE;                                                \
        if ((d_) == 0) fa_[0] = BM_LD(sp_ + fa_off[s_]);                                           \
        else if ((d_) <= NJ) fb_[((d_) - 1) % NJ] = BM_LD(sp_ + fb_off[s_] + BM_BOFF((d_) - 1));   \
        else fa_[((d_) - NJ) % RB] = BM_LD(sp_ + fa_off[s_] + ((d_) - NJ) * 1024);                 \
    }
#define BM_MFMA1(m_, fa_, fb_)                                                                     \
    {                                                                                              \
        if (DUAL)                                                                                  \
            asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0"                                          \
                : "+a"(acc[(m_) / NJ][(m_) % NJ]) : "v"(fa_[(m_) / NJ]), "v"(fb_[(m_) % NJ]));     \
        else                                                                                       \
            asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0"                                          \
                : "+a"(acc[(m_) / NJ][(m_) % NJ]) : "v"(fb_[(m_) % NJ]), "v"(fa_[(m_) / NJ]));     \
    }

    BM_LOOKUP(work.small0 + item);
    int load_item = item;
    BM_WAIT_VM_LGKM(0, 0);
    BM_ADOPT();
#pragma unroll
    for (int t = 0; t < NS; ++t)
#pragma unroll
        for (int j = 0; j < NL; ++j) BM_DMA(t, kbeg + t, j)
    int st = 0;                                        // stage of k-step kt
    BM_WAIT_VMCNT(NL * (NS - 1));
    for (;;) {
        const int t_row0 = row0, t_row_end = row_end, t_n0 = n0, t_n_end = n_end, t_tile = load_item;   // the tile being multiplied
        const int t_kbeg = kbeg, t_kend = kend;
        int n_kbeg, n_kend;
        BM_NEXT_ITEM(n_more, n_kbeg, n_kend);
        if (n_more) BM_LOOKUP(work.small0 + item);
        bool more = false;
        // The k-steps, on the first RBL_ row blocks: a tile of at most 64 rows leaves the others out of the matrix work, the
        // fragment reads and the write-out (not of the loads: the waits count them): what they do not draw lets the others
        // clock higher (layers, us: DeepSeek-shaped 32 tokens 83 -> 80, Qwen3-shaped 512 / 2048 tokens 159 272 -> 155 261).  The
        // narrow loop does without: its launches are short, and the larger kernel costs them as much as it gives.
#define BM_TILE(RBL_)                                                                                            \
    {                                                                                                                 \
        constexpr int NM = (RBL_) * NJ;                        /* MFMAs per k slice of 32 */                          \
        constexpr int NR = (RBL_) + NJ;                        /* fragment reads per k slice */                       \
        constexpr int RSTEP = NM >= 2 * NR ? 2 : 1;            /* MFMAs per fragment read */                          \
        static_assert(NR * RSTEP <= NM, "every fragment is read under the slice before its own");                     \
        f32x4 acc[RBL_][NJ];                                                                                          \
        _Pragma("unroll") for (int i = 0; i < (RBL_); ++i)                                                            \
            _Pragma("unroll") for (int j = 0; j < NJ; ++j)                                                            \
                _Pragma("unroll") for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.0f;                                    \
        asm volatile("s_nop 7" : "+a"(acc[0][0]));                                                                    \
        BM_BARE_BARRIER();                                                                                            \
        _Pragma("unroll") for (int d = 0; d < NR; ++d) BM_RD(d, f0a, f0b, st, 0)                                      \
        for (int kt = t_kbeg; kt < t_kend; ++kt) {                                                                    \
            const int kl = more ? kbeg + (kt + NS - t_kend) : kt + NS;                                                \
            const int stn = st == NS - 1 ? 0 : st + 1;                                                                \
            BM_WAIT_VM_LGKM(63, 0);                                                                                   \
            _Pragma("unroll") for (int m = 0; m < NM; ++m) {                                                          \
                BM_MFMA1(m, f0a, f0b);                                                                                \
                if (m % RSTEP == 0 && m / RSTEP < NR) BM_RD(m / RSTEP, f1a, f1b, st, 1)                               \
                __builtin_amdgcn_sched_barrier(0);                                                                    \
            }                                                                                                         \
            BM_WAIT_VM_LGKM(NL * (NS - 2), 0);                                                                        \
            BM_BARE_BARRIER();                                                                                        \
            _Pragma("unroll") for (int m = 0; m < NM; ++m) {                                                          \
                BM_MFMA1(m, f1a, f1b);                                                                                \
                _Pragma("unroll") for (int j = m * NL / NM; j < (m + 1) * NL / NM; ++j) BM_DMA(st, kl, j)             \
                if (m % RSTEP == 0 && m / RSTEP < NR) BM_RD(m / RSTEP, f0a, f0b, stn, 0)                              \
                __builtin_amdgcn_sched_barrier(0);                                                                    \
            }                                                                                                         \
            st = stn;                                                                                                 \
            if (kt == t_kend - NS - 1) {                                                                              \
                more = n_more;                                                                                        \
                if (more) {                                                                                           \
                    if (t_kend - t_kbeg < 2 * NS - 1) BM_WAIT_VM_LGKM(0, 0);                                          \
                    kbeg = n_kbeg; kend = n_kend; load_item = item;                                                   \
                    BM_ADOPT();                                                                                       \
                }                                                                                                     \
            }                                                                                                         \
        }                                                                                                             \
        /* last MFMA -> first access to an accumulator (see k64w_body).  Each loop has its own accumulators and its own */\
        /* write-out: joined behind the two loops, the compiler moves accumulators to other registers in front of */  \
        /* the wait, wherever it stands and whichever of them it is tied to */                                        \
        asm volatile("s_nop 15\n\ts_nop 15" : "+a"(acc[(RBL_) - 1][NJ - 1]));                                         \
        if (SPLIT && t_kend - t_kbeg < KT)                                                                            \
            store_partial<(RBL_), NJ>(partial_tile(p.splitk, work, xcd, work.nb - work.full + t_tile,                 \
                                                   work.piece_at(t_kbeg)) + wave * (RB * NJ * 256), acc, t_row0, t_row_end);\
        else                                                                                                          \
            k64s_write<DUAL, (RBL_), NJ>(acc, reinterpret_cast<uint32_t *>(smem + NS * STAGE) + wave * 1024, c, N, t_row0, t_row_end,\
                                         t_n0 + wave * (DUAL ? 8 : 16) * NJ, t_n_end, lane);                          \
    }
        if (NJ == 4 && t_row_end - t_row0 <= RB * 8) BM_TILE(RB / 2)
        else BM_TILE(RB)
#undef BM_TILE
        if (!more) break;
    }
    BM_WAIT_VM_LGKM(0, 0);
#undef BM_LOOKUP
#undef BM_NEXT_ITEM
#undef BM_ADOPT
#undef BM_DMA_AT
#undef BM_DMA
#undef BM_LD
#undef BM_BOFF
#undef BM_RD
#undef BM_MFMA1
}

// Both tile heights in one launch: p.mt_group / mt_row0 / n_mtiles list the 256-row tiles, p.mt_group_s / mt_row0_s /
// n_mtiles_s the 128-row tiles.
template <bool DUAL, bool SPLIT, bool MAY_STREAM>
__global__ void __launch_bounds__(256) grouped_gemm_mixed_k64w_bf16_kernel(GemmParams p) {
    const int n_nt = DUAL ? (p.N + 127) / 128 : (p.N + 255) / 256;
    XcdWork work;
    const SmallPlan plan(p.n_mtiles[0], small_tiles(p), n_nt, p.N / (DUAL ? 16 : 32), p.Kd / 64, K64_CUS, !SPLIT);
    work.init((p.n_mtiles[0] - plan.halved) * n_nt, (2 * plan.halved + small_tiles(p)) * plan.cols, p.Kd / 64, blockIdx.x & 7, SPLIT);
    if (SPLIT && blockIdx.x < K64_XCDS && threadIdx.x == 0) p.split_pieces[blockIdx.x] = work.S;
    // A 128-row tile is the only user of its weight panel (a group has at most one), so it streams from
    // memory at a third of a 256-row tile's arithmetic intensity.  When there are many of them (at least a
    // quarter of the 256-row tiles' number) every other workgroup takes its 128-row tiles first, so that the
    // streaming is spread over the launch instead of bunched at its end (Qwen3-shaped layer, 2048 tokens:
    // gate/up 141 -> 133 us); with few of them that order only delays 256-row tiles (Mixtral-shaped prefill
    // + 1 %, 1024 tokens + 3 %).
    // MAY_STREAM: all of the layer's groups together outgrow the memory-side cache; whether the live ones do is known here.  (Layers
    // that never do have a kernel without the second copies: 0.8 us of 50 in launches of short reductions.)
    // The cut down projection streams whatever the size of its weights: d = 1024 .. 2048, F = 4096 .. 5120, 50 to 130 MB, warm,
    // 200 to 1000 tokens: the same to 1 % either way.
    const bool stream = SPLIT || (MAY_STREAM && p.n_mtiles_s[2] > p.cached_groups);
    if (!SPLIT && plan.narrow) {
        if (stream) k64s_body<DUAL, SPLIT, true, 2>(p, work, plan);
        else k64s_body<DUAL, SPLIT, false, 2>(p, work, plan);
        return;
    }
    const bool small_first = small_tiles(p) * 4 >= p.n_mtiles[0] && ((blockIdx.x >> 3) & 1);
    const auto small = [&]() {
        if (stream) k64s_body<DUAL, SPLIT, true, 4>(p, work, plan);
        else k64s_body<DUAL, SPLIT, false, 4>(p, work, plan);
    };
    if (small_first) {
        small();
        __syncthreads();      // the last write-out's staging area becomes the next phase's first load target
        k64w_body<DUAL, SPLIT>(p, work);
    } else {
        k64w_body<DUAL, SPLIT>(p, work);
        __syncthreads();
        small();
    }
}

// Adds up the pieces of every cut tile of the down projection, in their order along the reduction, and writes the bf16 result.
// Grid 8 XCDs x 16 slices of a tile x cut tiles, the XCD fastest: workgroups are dealt round-robin to the XCDs, so a
// tile's pieces are read where they were written and partly still sit in that XCD's L2.  A workgroup handles one slice - four
// accumulator tiles of each of the writers' waves - with the writers' thread -> element mapping, so that the sums are
// spread over the chip.
__global__ void __launch_bounds__(256) split_fixup_kernel(GemmParams p) {
    const int xcd = blockIdx.x & 7, slice = (blockIdx.x >> 3) & 15, tile = blockIdx.x >> 7;
    const int n_nt = (p.N + 255) / 256, n_mt = p.n_mtiles[0];
    XcdWork work;
    const int n = p.split_pieces[xcd];                     // S, as the workgroups of the launch before chose it
    if (n == 1) return;
    work.init(n_mt * n_nt, small_tiles(p) * n_nt, p.Kd / 64, xcd, false);
    work.cut(n);
    const int R = work.nb - work.full;
    const bool big = tile < R;
    if (tile >= R + work.ns || (!big && slice >= 8)) return;
    int mt, nt;
    if (big) tile_of(work.big0 + work.full + tile, n_mt, n_nt, mt, nt);
    else { mt = (work.small0 + tile - R) / n_nt; nt = (work.small0 + tile - R) % n_nt; }
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r16 = lane & 15, quad = lane >> 4;
    const int g = big ? p.mt_group[mt] : p.mt_group_s[mt];
    const int i = big ? slice >> 1 : slice;                // row block inside the wave's part of the tile
    const int row0 = (big ? p.mt_row0[mt] + (wave >> 1) * 128 : p.mt_row0_s[mt]) + i * 16, row_end = p.offsets[g + 1], N = p.N;
    if (row0 >= row_end) return;
    const size_t ofs = (size_t)wave * (big ? 64 * 256 : 32 * 256) + (big ? i * 8 + (slice & 1) * 4 : i * 4) * 256 + lane * 4;
    // all loads go out before the first sum: one round trip to memory instead of one per piece
    f32x4 part[SPLIT_MAX][4];
#pragma unroll
    for (int c = 0; c < SPLIT_MAX; ++c)
        if (c < n) {
            const float *src = partial_tile(p.splitk, work, xcd, tile, c) + ofs;
#pragma unroll
            for (int q = 0; q < 4; ++q) part[c][q] = *(const BM_GLOBAL f32x4 *)(src + q * 256);
        }
    uint16_t *out = static_cast<uint16_t *>(p.c);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        f32x4 sum = part[0][q];
#pragma unroll
        for (int c = 1; c < SPLIT_MAX; ++c)
            if (c < n) sum += part[c][q];
        // transposed accumulator tiles: the lane holds columns 4 * quad .. + 3 of row r16
        const int col = nt * 256 + (big ? (wave & 1) * 128 + ((slice & 1) * 4 + q) * 16 : wave * 64 + q * 16) + 4 * quad;
        const int row = row0 + r16;
        if (row < row_end && col < N) {
            u32x2 pk;
            pk[0] = pack_bf16x2(sum[0], sum[1]);
            pk[1] = pack_bf16x2(sum[2], sum[3]);
            *(BM_GLOBAL u32x2 *)(&out[(size_t)row * N + col]) = pk;
        }
    }
}

static int grid_for(const GemmParams &p, bool dual) {
    const int n_nt = dual ? (p.N + 127) / 128 : (p.N + 255) / 256;
    const int total = p.max_mtiles * n_nt;
    return ((total + 7) / 8) * 8;
}

// compute units and XCDs of the current device (0, 0 if the queries fail)
static void device_shape(int &cus, int &xcds) {
    int dev = 0;
    cus = xcds = 0;
    if (hipGetDevice(&dev) != hipSuccess) return;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) cus = 0;
    if (hipDeviceGetAttribute(&xcds, hipDeviceAttributeNumberOfXccs, dev) != hipSuccess) xcds = 0;
}

bool persistent_device() {
    int cus, xcds;
    device_shape(cus, xcds);
    return persistent_schedule_fits(cus, xcds);
}

// the k-step-64 kernel addresses rows by 32-bit byte offsets from a uniform base, and its schedule is laid
// out for the full part (see bm_device_shape.h)
static bool k64_ok(const GemmParams &p) {
    const unsigned long long lim = 1ull << 32;
    if (!persistent_device()) return false;
    // (and hands the loads over to the next tile three k-steps before a tile ends)
    return p.BM == 256 && p.Kd % 64 == 0 && p.Kd >= 256 && (unsigned long long)p.a_rows * p.Kd * 2 < lim &&
           (unsigned long long)p.N * p.Kd * 2 < lim;
}

template <bool DUAL>
static void launch_mixed(const GemmParams &p, hipStream_t st) {
    if (p.n_groups > p.cached_groups)
        hipLaunchKernelGGL((grouped_gemm_mixed_k64w_bf16_kernel<DUAL, false, true>), dim3(K64_CUS), dim3(256), 0, st, p);
    else
        hipLaunchKernelGGL((grouped_gemm_mixed_k64w_bf16_kernel<DUAL, false, false>), dim3(K64_CUS), dim3(256), 0, st, p);
}

int launch_gateup_bf16(const GemmParams &p, hipStream_t st) {
    if (p.mixed && k64_ok(p))
        launch_mixed<true>(p, st);
    else if (p.mixed)
        return -1;                // the caller asks for both tile heights only where the persistent kernel runs
    else if (p.BM == 256)
        hipLaunchKernelGGL((grouped_gemm256_dma_bf16_kernel<true>), dim3(grid_for(p, true)), dim3(256), 0, st, p);
    else
        hipLaunchKernelGGL((grouped_gemm_bf16_kernel<true, 128>), dim3(grid_for(p, true)), dim3(256), 0, st, p);
    return launch_status(__func__);
}

// cutting tiles along the reduction (see XcdWork) pays only for long reductions
bool down_split_tail(int Kd) { return Kd / 64 >= 64; }

int launch_down_bf16(const GemmParams &p, hipStream_t st) {
    if (p.BM == 256 && k64_ok(p) && p.splitk != nullptr && down_split_tail(p.Kd)) {
        hipLaunchKernelGGL((grouped_gemm_mixed_k64w_bf16_kernel<false, true, true>), dim3(K64_CUS), dim3(256), 0, st, p);
        const int tiles = p.mixed ? FIXUP_TILES : FIXUP_TILES_256;
        hipLaunchKernelGGL(split_fixup_kernel, dim3(K64_XCDS * 16 * tiles), dim3(256), 0, st, p);
    } else if (p.mixed && k64_ok(p)) {
        launch_mixed<false>(p, st);
    } else if (p.mixed) {
        return -1;
    } else if (p.BM == 256) {
        hipLaunchKernelGGL((grouped_gemm256_dma_bf16_kernel<false>), dim3(grid_for(p, false)), dim3(256), 0, st, p);
    } else {
        hipLaunchKernelGGL((grouped_gemm_bf16_kernel<false, 128>), dim3(grid_for(p, false)), dim3(256), 0, st, p);
    }
    return launch_status(__func__);
}

}  // namespace bm
