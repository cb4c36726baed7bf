// Products of the 128 rows of a panel with the rows of a tall matrix, over fp16 terms (v_mfma_f32_16x16x32_f16, fp32 sums):
//     C = Y X^T   or   C -= Y X^T,     Y: 128 x K, X: N x K, both k-contiguous fp32, N a multiple of 128, K of 32
// the two halves of the projection of a panel against the finished rows in the SOAP refresh.  Both operands are scaled by
// powers of two and cut into NY and NX fp16 terms (2: 22 bits) on the way; terms that are not made are not multiplied.
//
// A workgroup of 4 wavefronts takes 64 MI rows of X, 16 MI of them per wavefront, and all of Y.  The rows of X belong to one
// wavefront, so they go from memory straight into the lanes that multiply them and are cut there; Y, which all share, goes
// through two LDS stages.  An X row's terms pass once through registers for 128 products instead of through LDS: with
// both operands staged, as in gemm_bf16.h, a 128 x 128 tile needs as many LDS cycles as matrix cycles.  What bounds the refresh's
// products now is memory: every panel reads all finished rows (n = 2048, 636 factors, the 15th panel: 9.3 GB in 2.0 ms), so
// where `panels` > 1 several panels share one pass over them; the tiles that do run side by side on one XCD.
// Refresh of the 1.1B model (gemm_bf16.h: 135.0 ms): 128.3; with two panels a pass in the first sweep 123.1.
#pragma once
#include "gemm.h"
#include "gemm_bf16.h"
#include "pgemm.h"

namespace asteria {

constexpr int PP_ROWS = 128, PP_BK = 32;

struct PanelProblem {
    const float *X, *Y;
    float *C;
    const float *y_scale;    // on the device; X is scaled by x_scale
    float x_scale;
    int N, K, ldx, ldy, ldc;
    int state_idx;           // runs while the state word at this index is 0
    int subtract;
    int panels;              // Y and C: this many panels of 128 rows ...
    int slots;               // ... of `slots` tiles per tile of X
    int start[2];            // first tile of 128, of 256 rows of X
};

constexpr size_t pp_lds_bytes(int ny) { return 2u * PP_ROWS * 64u * (size_t)ny; }

// tile t_global of a launch, 256 threads; pp_lds_bytes at smem_raw
// YR: rows of Y, part `part` of the panel's 128
template <int NY, int NX, int MI, int YR = PP_ROWS>
__device__ __forceinline__ void panel_product_tile(const PanelProblem *__restrict__ probs, int nprobs, int t_global, const int *__restrict__ state,
                                                   unsigned char *smem_raw, int part = 0)
{
    constexpr int NJ = YR / 16, TX = 64 * MI, WSEL = MI == 4 ? 1 : 0, NV = YR / 32;    // NV: loads of Y per wavefront and slab
    constexpr uint32_t ROWB = 64u * NY, STAGE = YR * ROWB;
    typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
    ASTERIA_LDS char *lds = (ASTERIA_LDS char *)smem_raw;
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
    int plo = 0, phi = nprobs - 1;
    while (plo < phi) {
        const int mid = (plo + phi + 1) >> 1;
        if (probs[mid].start[WSEL] <= t_global) plo = mid; else phi = mid - 1;
    }
    const PanelProblem P = probs[plo];
    if (state[P.state_idx] != 0) return;
    // the panels of a tile of X are neighbours on one XCD: its rows come from memory once
    const int lt = t_global - P.start[WSEL], panel = lt % P.slots;
    if (panel >= P.panels) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int x0 = (lt / P.slots) * TX + wave * (16 * MI), nk = P.K / PP_BK;
    const float scx = P.x_scale, scy = uniform(*P.y_scale);

    // ---- Y: memory -> registers -> LDS.  A load instruction brings 8 rows of 32 values, a wavefront its quarter of the rows.  An LDS row is
    // [32 hi][32 lo] in 16-byte chunks swizzled by row; chunk g holds k = 4 g .. 4 g + 3 and 16 + 4 g .. 19 + 4 g, as X does
    const char *gy = reinterpret_cast<const char *>(P.Y) + (size_t)(panel * PP_ROWS + part * YR + wave * (YR / 4)) * P.ldy * 4;
    const uint32_t vy = (uint32_t)(lane >> 3) * (uint32_t)P.ldy * 4u + (uint32_t)(lane & 7) * 16u;
    const size_t sy = (size_t)P.ldy * 32;
    u32x4 ry[NV];
    auto load_y = [&](int s) __attribute__((always_inline)) {
        const size_t slab = (size_t)min(s, nk - 1);
#pragma unroll
        for (int v = 0; v < NV; ++v) ry[v] = *(const ASTERIA_GLOBAL u32x4 *)(gy + (v * sy + slab * 128) + vy);
    };
    const uint32_t wrow = lds0 + (uint32_t)(wave * (YR / 4) + (lane >> 3)) * ROWB + (uint32_t)((lane >> 2) & 1) * 8u;
    const uint32_t wy = wrow + (uint32_t)((NY == 2 ? (lane & 3) ^ (lane >> 4) : (lane & 3) ^ (lane >> 5)) * 16);
    auto split = [](u32x4 x, float scale, uint32_t (&hi)[2], uint32_t (&lo)[2]) __attribute__((always_inline)) {
        pg_split_f16(__uint_as_float(x[0]), __uint_as_float(x[1]), scale, hi[0], lo[0]);
        pg_split_f16(__uint_as_float(x[2]), __uint_as_float(x[3]), scale, hi[1], lo[1]);
    };
    auto stage = [&](uint32_t o, int v) __attribute__((always_inline)) {
        uint32_t hi[2], lo[2];
        split(ry[v], scy, hi, lo);
        const uint32_t at = (((YR == 32 ? wave : v) & 1) ? (wy + o) ^ (NY == 2 ? 64u : 32u) : wy + o);   // rows 8 on: the swizzle's top bit
        *(ASTERIA_LDS u32x2_t *)(uintptr_t)(at + v * (8 * ROWB)) = (u32x2_t){hi[0], hi[1]};
        if constexpr (NY == 2) *(ASTERIA_LDS u32x2_t *)(uintptr_t)((at ^ 64u) + v * (8 * ROWB)) = (u32x2_t){lo[0], lo[1]};
    };
    auto lds_barrier = []() __attribute__((always_inline)) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
    };
    load_y(0);
#pragma unroll
    for (int v = 0; v < NV; ++v) stage(0, v);
    load_y(1);

    // wavefronts beyond the last row of X stage their part of Y and leave
    if (x0 >= P.N) {
        uint32_t o = STAGE;
        lds_barrier();
        for (int kt = 0; kt < nk; ++kt) {
#pragma unroll
            for (int v = 0; v < NV; ++v) stage(o, v);
            load_y(kt + 2);
            o ^= STAGE;
            lds_barrier();
        }
        lds_barrier();
        return;
    }

    // ---- X: memory -> registers, 16 rows an instruction, four lanes 64 bytes of a row
    const int r16 = lane & 15, g16 = lane >> 4;
    const char *gx = reinterpret_cast<const char *>(P.X) + (size_t)x0 * P.ldx * 4;
    const uint32_t vx = (uint32_t)r16 * (uint32_t)P.ldx * 4u + (uint32_t)g16 * 16u;
    const size_t sx = (size_t)P.ldx * 64;
    u32x4 rx[MI][2], xh[MI], xl[MI], y[2][NY];
    auto load_x = [&](int s) __attribute__((always_inline)) {
        const size_t slab = (size_t)min(s, nk - 1);
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            rx[i][0] = *(const ASTERIA_GLOBAL u32x4 *)(gx + (i * sx + slab * 128) + vx);
            rx[i][1] = *(const ASTERIA_GLOBAL u32x4 *)(gx + (i * sx + slab * 128 + 64) + vx);
        }
    };
    auto split_x = [&](int i) __attribute__((always_inline)) {
        uint32_t h0[2], l0[2], h1[2], l1[2];
        split(rx[i][0], scx, h0, l0);
        split(rx[i][1], scx, h1, l1);
        xh[i] = (u32x4){h0[0], h0[1], h1[0], h1[1]};
        if constexpr (NX == 2) xl[i] = (u32x4){l0[0], l0[1], l1[0], l1[1]};
    };
    const uint32_t fy = lds0 + (uint32_t)r16 * ROWB + (NY == 2 ? (uint32_t)((g16 ^ ((r16 >> 1) & 7)) * 16) : (uint32_t)((g16 ^ ((r16 >> 2) & 3)) * 16));
    uint32_t o = 0;                                   // stage being read
    auto read_y = [&](int q, int j) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < NY; ++t) y[q][t] = *(const ASTERIA_LDS u32x4 *)(uintptr_t)(((fy + o) ^ (t ? 64u : 0u)) + j * (16 * ROWB));
    };
    // D = X rows x Y rows: a lane holds 4 consecutive columns of one row of C
    auto mma = [](u32x4 a, u32x4 b, floatx4 c) __attribute__((always_inline)) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(pg_f16x8, a), __builtin_bit_cast(pg_f16x8, b), c, 0, 0, 0);
    };
    floatx4 acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = (floatx4){0.0f, 0.0f, 0.0f, 0.0f};
    load_x(0);
#pragma unroll
    for (int i = 0; i < MI; ++i) split_x(i);
    load_x(1);
    lds_barrier();
    read_y(0, 0);
    for (int kt = 0; kt < nk; ++kt) {
        const uint32_t no = o ^ STAGE;
        // all column blocks but the last: small cross terms first, the leading product last
#pragma unroll
        for (int j = 0; j + 1 < NJ; ++j) {
            const int q = j & 1;
            read_y(q ^ 1, j + 1);
            if constexpr (NX == 2)
#pragma unroll
                for (int i = 0; i < MI; ++i) acc[i][j] = mma(xl[i], y[q][0], acc[i][j]);
            if constexpr (NY == 2)
#pragma unroll
                for (int i = 0; i < MI; ++i) acc[i][j] = mma(xh[i], y[q][1], acc[i][j]);
#pragma unroll
            for (int i = 0; i < MI; ++i) acc[i][j] = mma(xh[i], y[q][0], acc[i][j]);
            if (j < NV) stage(no, j);
            if (j == (NV < NJ - 2 ? NV : NJ - 2)) load_y(kt + 2);
            __builtin_amdgcn_sched_barrier(0);
        }
        // the last one: the next slab is staged and everyone has read this one; two row blocks at a time, whose lanes then take
        // the next slab's values
        constexpr int j = NJ - 1, q = j & 1;
        lds_barrier();
        o = no;
        read_y(q ^ 1, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < MI; i += 2) {
            if constexpr (NX == 2) { acc[i][j] = mma(xl[i], y[q][0], acc[i][j]); acc[i + 1][j] = mma(xl[i + 1], y[q][0], acc[i + 1][j]); }
            if constexpr (NY == 2) { acc[i][j] = mma(xh[i], y[q][1], acc[i][j]); acc[i + 1][j] = mma(xh[i + 1], y[q][1], acc[i + 1][j]); }
            acc[i][j] = mma(xh[i], y[q][0], acc[i][j]);
            acc[i + 1][j] = mma(xh[i + 1], y[q][0], acc[i + 1][j]);
            __builtin_amdgcn_sched_barrier(0);
            split_x(i);
            split_x(i + 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        load_x(kt + 2);
    }

    // ---- stores: 32 x 32 through 4 KiB per wavefront, whole 128-byte row pieces
    lds_barrier();
    const float inv = 1.0f / (scx * scy);             // powers of two: exact
    ASTERIA_LDS char *ws = lds + wave * 4096;
    int ln = lane;
    asm volatile("" : "+v"(ln));                     // addresses are made here, not kept through the K loop
    const int rr = ln >> 3, e8 = ln & 7;
    ASTERIA_GLOBAL float *C = (ASTERIA_GLOBAL float *)P.C + (size_t)(panel * PP_ROWS + part * YR + rr) * P.ldc + x0 + 4 * e8;
#pragma unroll
    for (int jj = 0; jj < NJ / 2; ++jj)
#pragma unroll
        for (int ii = 0; ii < MI / 2; ++ii) {
            ASTERIA_GLOBAL float *c = C + (size_t)(32 * jj) * P.ldc + 32 * ii;
            floatx4 old[4];
            if (P.subtract) {
#pragma unroll
                for (int p = 0; p < 4; ++p) old[p] = *(const ASTERIA_GLOBAL floatx4 *)(c + (size_t)(8 * p) * P.ldc);
            }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int w = 0; w < 2; ++w) {
                    const int r = 16 * u + (ln & 15);
                    *(ASTERIA_LDS floatx4 *)(ws + r * 128 + (((4 * w + (ln >> 4)) ^ (r & 7)) * 16)) = acc[2 * ii + w][2 * jj + u];
                }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const int r = p * 8 + rr;
                floatx4 t = *(const ASTERIA_LDS floatx4 *)(ws + r * 128 + ((e8 ^ (r & 7)) * 16));
#pragma unroll
                for (int e = 0; e < 4; ++e) t[e] = P.subtract ? fmaf(-inv, t[e], old[p][e]) : inv * t[e];
                *(ASTERIA_GLOBAL floatx4 *)(c + (size_t)(8 * p) * P.ldc) = t;
            }
        }
}

template <int NY, int NX, int MI, int YR = PP_ROWS>
__global__ __launch_bounds__(256, 2) void panel_product_kernel(const PanelProblem *__restrict__ probs, int nprobs, int total_tiles,
                                                               const int *__restrict__ state)
{
    constexpr int PARTS = PP_ROWS / YR;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int total = PARTS * total_tiles, per_xcd = (total + NUM_XCD - 1) / NUM_XCD;
    const int t = (int)(blockIdx.x % NUM_XCD) * per_xcd + (int)(blockIdx.x / NUM_XCD);
    if (t < total) panel_product_tile<NY, NX, MI, YR>(probs, nprobs, t / PARTS, state, smem_raw, t % PARTS);
}

// `tiles` tiles of whole panels and the tiles of gemm_bf16.h of panels with a remainder, in one launch.  Either kind is spread over
// the XCDs (joint_tile); the slower ones, with guards, come first.  SOAP refresh in us, joint / apart: matrices of 899 x 1405 in blocks of
// 256 (38 of 256, 6 of 131, 4 of 125 each), 1: 685 / 768, 5: 809 / 929, 20: 1720 / 1869, 50: 4551 / 4705; of 1100 x 1405 in blocks of 512, 4: 1441
// / 1574, 50: 5627 / 5853; of 1100 x 2500 in blocks of 1024, 4: 3165 / 3454, 40: 12409 / 12764.
template <int NY, int NX, int MI, bool PARTS = false>
__global__ __launch_bounds__(256, 2) void joint_product_kernel(const PanelProblem *__restrict__ probs, int nprobs, int tiles,
                                                               const GemmProblem *__restrict__ ragged, int nragged, int ragged_tiles,
                                                               const int *__restrict__ state)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    constexpr int P = PARTS ? 4 : 1;
    bool second;
    const int t = joint_tile(P * ragged_tiles, P * tiles, second);
    if (t < 0) return;
    if (second) panel_product_tile<NY, NX, MI, PP_ROWS / P>(probs, nprobs, t / P, state, smem_raw, t % P);
    else gemm_bf16_tile<float, float, NY, NX, true, PARTS>(ragged, nragged, t / P, state, smem_raw, t % P);
}

// Whether a launch takes 256 rows of X per tile (MI = 4) or 128 (MI = 2: 150 registers, three workgroups on a CU);
// `tiles_256`: tiles of 256.  The large ones read and cut Y half as often but pay only once two of them are on every CU.
// SOAP refresh on small over large tiles: 8 factors of n = 2048 0.83, 32: 1.00, 48 (384 tiles of the second product): 0.99,
// 64 (512): 1.015, 96: 1.02, 192: 1.03; n = 1024, 32 factors 0.91, 128: 1.00, 256 (1024 tiles): 1.00; n = 512, 64: 0.94,
// 256: 1.01; n = 256, 256: 0.98, 1024 (1024 tiles): 0.96.
inline bool pp_take_wide_tiles(int tiles_256)
{
    return tiles_256 >= 512;
}

// Few tiles of 128 rows of X: a quarter of the panel's rows per workgroup, whose products of a slab take less time than its loads.  The
// sums of an element and their order stay.  SOAP refresh in us, whole / quarters up to 64 tiles / up to 128: 1 factor of n = 2048 (and 256) 5571
// / 5131 / 5129, 4 of 640 and 1024 2133 / 2068 / 2067, 16 of 1024 2497 / 2368 / 2415, 32 of 1024 2772 / 2691 / 2875, 20 of 512 and 384 1040 /
// 1008 / 1017.  Launches of both kinds of tiles, up to 200 (whose guarded tiles wait longest): whole / quarters, 1 matrix of 899 x 1405 in
// blocks of 1024 2694 / 2160, of 256 902 / 802, 4 of 1100 x 2500 4740 / 4420 (up to 64: 4638), 4 of 1100 x 1405 in blocks of 512 1264 / 1176, 10 of
// 1300 x 1500 3319 / 3228, 20 of 600 x 400 1215 / 1120.
constexpr int PP_PART_TILES = 64, PP_JOINT_TILES = 200;

template <int NY, int NX, int MI>
inline hipError_t launch_panel_product(const PanelProblem *probs, int nprobs, int total_tiles, const int *state, hipStream_t stream)
{
    if (total_tiles <= 0 || nprobs <= 0) return hipSuccess;
    constexpr size_t lds = pp_lds_bytes(NY);
    const bool parts = MI == 2 && total_tiles <= PP_PART_TILES;
    const int per_xcd = ((parts ? 4 : 1) * total_tiles + NUM_XCD - 1) / NUM_XCD;
    auto kern = parts ? panel_product_kernel<NY, NX, 2, PP_ROWS / 4> : panel_product_kernel<NY, NX, MI>;
    profile_begin(515, stream);
    hipLaunchKernelGGL(kern, dim3(per_xcd * NUM_XCD), dim3(256), lds, stream, probs, nprobs, total_tiles, state);
    profile_end(stream);
    return hipGetLastError();
}

template <int NY, int NX, int MI>
inline hipError_t launch_joint_product(const PanelProblem *probs, int nprobs, int tiles, const GemmProblem *ragged, int nragged, int ragged_tiles,
                                       const int *state, hipStream_t stream)
{
    if (tiles + ragged_tiles <= 0) return hipSuccess;
    const bool parts = MI == 2 && tiles + ragged_tiles <= PP_JOINT_TILES;
    auto kern = parts ? joint_product_kernel<NY, NX, 2, true> : joint_product_kernel<NY, NX, MI>;
    constexpr size_t lds = gemm_bf16_lds<float, float, NY, NX>();
    static_assert(lds >= pp_lds_bytes(NY), "either kind of tile");
    static bool configured[2][MAX_DEVICES] = {};
    if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kern), lds, configured[parts]); e != hipSuccess) return e;
    const int p = parts ? 4 : 1;
    profile_begin(515, stream);
    hipLaunchKernelGGL(kern, dim3(joint_grid(p * ragged_tiles, p * tiles)), dim3(256), lds, stream, probs, nprobs, tiles, ragged, nragged,
                       ragged_tiles, state);
    profile_end(stream);
    return hipGetLastError();
}

}  // namespace asteria
