// Guard-free grouped GEMM over 16-bit terms on the gfx950 matrix cores (v_mfma_f32_16x16x32, fp32 accumulation).
//
// One launch walks a device table of problems  C = A B^T  (A is M x K, B is N x K, both k-contiguous, M and N whole
// tiles, K a multiple of 32: the callers send other shapes to the guarded kernels).  A is a plain fp32 matrix that the loader cuts into two
// bf16 terms (the value rounded, the remainder rounded) while it stages it; B is the same (NTB = 2: three products per
// block, lo hi, hi lo, hi hi, 16 bits of both operands) or a plain bf16 matrix (NTB = 1: two products).  With F16 the terms
// are fp16 ones (22 bits) of the operands times powers of two that the problem states.
#pragma once
#include <type_traits>

#include "gemm.h"

namespace asteria {

typedef __bf16 pg_bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 pg_f16x8 __attribute__((ext_vector_type(8)));

struct PlaneProblem {
    const void *A;          // fp32 matrix
    const void *B;          // fp32 or bf16 matrix
    float *C32;             // fp32 output (GEMM_C_BF16: a bf16 matrix)
    int M, N, K;
    int lda, ldb, ldc32;    // elements
    int tile_start;
    int tiles_n;            // tile columns
    int flags;
    float sa, sb;           // fp16 terms: powers of two the operands are multiplied by before the split,
    const float *sa_dev, *sb_dev;   // on the device where these are not null
};

__device__ __forceinline__ uint32_t pg_pack_bf16(float a, float b)
{
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    typedef float floatx2_t __attribute__((ext_vector_type(2)));
    const floatx2_t f = {a, b};                  // as a vector: one v_cvt_pk_bf16_f32 (round to nearest even)
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));
}

// two fp16 terms of (a, b) * scale, round to nearest in both; scale is a power of two, so the fused product is exact
__device__ __forceinline__ void pg_split_f16(float a, float b, float scale, uint32_t &hi, uint32_t &lo)
{
    typedef _Float16 halfx2_t __attribute__((ext_vector_type(2)));
    typedef float floatx2_t __attribute__((ext_vector_type(2)));
    const halfx2_t h = __builtin_convertvector(((floatx2_t){a * scale, b * scale}), halfx2_t);
    const floatx2_t d = {fmaf(a, scale, -(float)h[0]), fmaf(b, scale, -(float)h[1])};
    hi = __builtin_bit_cast(uint32_t, h);
    lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(d, halfx2_t));
}

// A 256 x 256 tile per workgroup of 8 wavefronts (4 x 2), 64 x 128 each in MFMA blocks of 16 x 16; slabs of 32 k, two stages.
// An LDS row holds 32 k of a matrix row: [32 hi][32 lo] (128 bytes, 16-byte chunks swizzled by row) or 32 bf16 (64 bytes).
// A slab is loaded into registers a slab ahead, cut into terms and stored behind the products of the slab before its own; the
// barrier between two slabs comes before the last column block, behind whose products the next slab's first operands
// are read.  So the matrix pipe waits for neither: before this, two groups of wavefronts alternated between fragment reads
// and products at a barrier each (pipe busy 47 - 49 %).
// Measured (this kernel, the one before): preconditioned update of the 1.1B model 10.0 ms, 12.2; SOAP step 43.9 ms, 52.6 (four
// rotations, Adam 5.0 of it).  SOAP refresh of that model with its products A Q here (F16), on the 128 x 128 tiles of gemm_bf16.h:
// 135.0 ms, 147.3.
// TILE = 128: 4 wavefronts (2 x 2) of 64 x 64, two workgroups on a CU, for launches too small for the large tiles.  Every element has
// the same sums in the same order, so which of the two a launch takes does not show in its result.
constexpr int PG_TILE = 256, PG_SMALL_TILE = 128, PG_BK = 32;
constexpr size_t pg_lds_bytes(int ntb, int tile) { return 2u * (size_t)tile * (128 + 64 * ntb); }

// tile t_global of a launch, 2 TILE threads; pg_lds_bytes at smem_raw
template <int NTB, bool F16, int TILE>
__device__ __forceinline__ void pgemm_tile(const PlaneProblem *__restrict__ probs, int nprobs, int t_global, unsigned char *smem_raw)
{
    constexpr int MI = 4, NJ = TILE / 32;
    static_assert(NJ == 8 || NJ == 4, "two columns of wavefronts, 64 rows each; four pieces to stage behind NJ - 1 blocks");
    constexpr uint32_t ROWB = 64u * NTB, STAGE_A = TILE * 128u, STAGE_B = TILE * ROWB;
    typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
    ASTERIA_LDS char *lds = (ASTERIA_LDS char *)smem_raw;
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
    int plo = 0, phi = nprobs - 1;
    while (plo < phi) {
        const int mid = (plo + phi + 1) >> 1;
        if (probs[mid].tile_start <= t_global) plo = mid; else phi = mid - 1;
    }
    const PlaneProblem P = probs[plo];   // by value: the fields stay in scalar registers across the stores below
    const int lt = t_global - P.tile_start, ti = lt / P.tiles_n, tj = lt % P.tiles_n;
    const int row0 = ti * TILE, col0 = tj * TILE, nk = P.K / PG_BK;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    // ---- memory -> registers -> LDS.  A load instruction brings 8 rows of 32 fp32 (lane / 8 the row, lane % 8 four values) or 16
    // rows of 32 bf16; a wavefront its 32 rows of either operand
    const char *ga = reinterpret_cast<const char *>(P.A) + (size_t)(row0 + wave * 32) * P.lda * 4;
    const char *gb = reinterpret_cast<const char *>(P.B) + (size_t)(col0 + wave * 32) * P.ldb * (NTB == 2 ? 4 : 2);
    const uint32_t va = (uint32_t)(lane >> 3) * (uint32_t)P.lda * 4u + (uint32_t)(lane & 7) * 16u;
    const uint32_t vb = NTB == 2 ? (uint32_t)(lane >> 3) * (uint32_t)P.ldb * 4u + (uint32_t)(lane & 7) * 16u
                                 : (uint32_t)(lane >> 2) * (uint32_t)P.ldb * 2u + (uint32_t)(lane & 3) * 16u;
    const size_t sa = (size_t)P.lda * 32, sb = (size_t)P.ldb * 32;           // bytes of 8 fp32 rows, of 16 bf16 rows
    constexpr int NB = NTB == 2 ? 4 : 2;
    u32x4 ra[4], rb[NB];
    auto gload = [&](int s) __attribute__((always_inline)) {
        const size_t slab = (size_t)min(s, nk - 1);
#pragma unroll
        for (int v = 0; v < 4; ++v) ra[v] = *(const ASTERIA_GLOBAL u32x4 *)(ga + (v * sa + slab * 128) + va);
#pragma unroll
        for (int v = 0; v < NB; ++v) rb[v] = *(const ASTERIA_GLOBAL u32x4 *)(gb + (v * sb + slab * (NTB == 2 ? 128 : 64)) + vb);
    };
    // chunk (lane % 8) / 2 of the hi half; odd instructions are 8 rows on, which flips the swizzle's top bit
    const uint32_t wa = lds0 + (uint32_t)(wave * 32 + (lane >> 3)) * 128u + (uint32_t)((((lane & 7) >> 1) ^ (lane >> 4)) * 16 + (lane & 1) * 8);
    const uint32_t wb = NTB == 2 ? wa + 2 * STAGE_A
                                 : lds0 + 2 * STAGE_A + (uint32_t)(wave * 32 + (lane >> 2)) * 64u + (uint32_t)(((lane & 3) ^ ((lane >> 4) & 3)) * 16);
    float sca = 1.0f, scb = 1.0f;
    if (F16) { sca = uniform(P.sa_dev ? *P.sa_dev : P.sa); scb = uniform(P.sb_dev ? *P.sb_dev : P.sb); }
    auto split_store = [&](uint32_t at, u32x4 x, int v, float scale) __attribute__((always_inline)) {
        const float x0 = __uint_as_float(x[0]), x1 = __uint_as_float(x[1]), x2 = __uint_as_float(x[2]), x3 = __uint_as_float(x[3]);
        uint32_t h0, h1, l0, l1;
        if constexpr (F16) {
            pg_split_f16(x0, x1, scale, h0, l0);
            pg_split_f16(x2, x3, scale, h1, l1);
        } else {
            h0 = pg_pack_bf16(x0, x1); h1 = pg_pack_bf16(x2, x3);
            l0 = pg_pack_bf16(x0 - __uint_as_float(h0 << 16), x1 - __uint_as_float(h0 & 0xffff0000u));
            l1 = pg_pack_bf16(x2 - __uint_as_float(h1 << 16), x3 - __uint_as_float(h1 & 0xffff0000u));
        }
        const uint32_t hi = (v & 1) ? at ^ 64u : at;
        *(ASTERIA_LDS u32x2_t *)(uintptr_t)(hi + v * 1024) = (u32x2_t){h0, h1};
        *(ASTERIA_LDS u32x2_t *)(uintptr_t)((hi ^ 64u) + v * 1024) = (u32x2_t){l0, l1};
    };
    // piece q of 4 of the loaded slab
    auto stage = [&](uint32_t oa, uint32_t ob, int q) __attribute__((always_inline)) {
        split_store(wa + oa, ra[q], q, sca);
        if constexpr (NTB == 2) split_store(wb + ob, rb[q], q, scb);
        else if (q < 2) *(ASTERIA_LDS u32x4 *)(uintptr_t)(wb + ob + q * 1024) = rb[q];
    };

    // ---- LDS -> registers -> products
    const int r16 = lane & 15, g16 = lane >> 4;
    const uint32_t fch = (uint32_t)((g16 ^ ((r16 >> 1) & 7)) * 16);
    const uint32_t fa = lds0 + (uint32_t)(wm * 64 + r16) * 128u + fch;
    const uint32_t fb = lds0 + 2 * STAGE_A + (uint32_t)(wn * 16 * NJ + r16) * ROWB + (NTB == 2 ? fch : (uint32_t)((g16 ^ ((r16 >> 2) & 3)) * 16));
    auto frag = [](uint32_t p) __attribute__((always_inline)) { return *(const ASTERIA_LDS u32x4 *)(uintptr_t)p; };
    // D = B-rows x A-rows: a lane holds 4 consecutive columns of one row of C
    auto mma = [](u32x4 a, u32x4 b, floatx4 c) __attribute__((always_inline)) {
        if constexpr (F16)
            return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(pg_f16x8, b), __builtin_bit_cast(pg_f16x8, a), c, 0, 0, 0);
        else return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(pg_bf16x8, b), __builtin_bit_cast(pg_bf16x8, a), c, 0, 0, 0);
    };
    floatx4 acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = (floatx4){0.0f, 0.0f, 0.0f, 0.0f};
    u32x4 ah[MI], al[MI], b[2][NTB];
    uint32_t oa = 0, ob = 0;                          // stage being read
    auto read_a = [&](u32x4 (&d)[MI], uint32_t term) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < MI; ++i) d[i] = frag(((fa + oa) ^ term) + i * 2048);
    };
    auto read_b = [&](int q, int j) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < NTB; ++t) b[q][t] = frag(((fb + ob) ^ (t ? 64u : 0u)) + j * (16 * ROWB));
    };
    auto lds_barrier = []() __attribute__((always_inline)) {       // waits for LDS, not for the loads of the slab after next
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
    };
    gload(0);
#pragma unroll
    for (int q = 0; q < 4; ++q) stage(0, 0, q);
    gload(1);
    lds_barrier();
    read_a(al, 64u); read_a(ah, 0u); read_b(0, 0);
    for (int kt = 0; kt < nk; ++kt) {
        const uint32_t na = oa ^ STAGE_A, nb = ob ^ STAGE_B;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int q = j & 1;
            const bool end = j + 1 == NJ;
            if (!end) read_b(q ^ 1, j + 1);
            else {
                lds_barrier();                        // the next slab is staged, and everyone has read this one
                oa = na; ob = nb;
                read_b(q ^ 1, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            // small cross terms first, the leading product last
#pragma unroll
            for (int i = 0; i < MI; ++i) acc[i][j] = mma(al[i], b[q][0], acc[i][j]);
            if (end) { __builtin_amdgcn_sched_barrier(0); read_a(al, 64u); __builtin_amdgcn_sched_barrier(0); }
            if constexpr (NTB == 2)
#pragma unroll
                for (int i = 0; i < MI; ++i) acc[i][j] = mma(ah[i], b[q][1], acc[i][j]);
#pragma unroll
            for (int i = 0; i < MI; ++i) acc[i][j] = mma(ah[i], b[q][0], acc[i][j]);
            if (NJ == 8 ? j < 4 : j == 0) stage(na, nb, j);
            if (NJ == 4 && j < 3) stage(na, nb, j + 1);
            if (j == (NJ == 8 ? 4 : 2)) gload(kt + 2);
            __builtin_amdgcn_sched_barrier(0);
        }
        read_a(ah, 0u);
    }

    // ---- stores: 32 x 32 through 4 KiB per wavefront, whole 128-byte (bf16: 64-byte) row pieces
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    if constexpr (F16) {
        const float inv = 1.0f / (sca * scb);       // powers of two: exact
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[i][j] *= inv;
    }
    ASTERIA_LDS char *ws = lds + wave * 4096;
    const bool bf16 = (P.flags & GEMM_C_BF16) != 0;
    const bool vec = (P.ldc32 & 3) == 0 && (reinterpret_cast<uintptr_t>(P.C32) & (bf16 ? 7u : 15u)) == 0;
    int ln = lane;
    asm volatile("" : "+v"(ln));                    // addresses are made here, not kept through the K loop
    const int rr = ln >> 3, e8 = ln & 7;
#pragma unroll
    for (int i = 0; i < MI / 2; ++i)
#pragma unroll
        for (int j = 0; j < NJ / 2; ++j) {
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int w = 0; w < 2; ++w) {
                    const int r = 16 * u + (ln & 15);
                    *(ASTERIA_LDS floatx4 *)(ws + r * 128 + (((4 * w + (ln >> 4)) ^ (r & 7)) * 16)) = acc[2 * i + u][2 * j + w];
                }
            __builtin_amdgcn_wave_barrier();
            const int br = row0 + wm * 64 + i * 32, bc = col0 + wn * 16 * NJ + j * 32 + 4 * e8;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = q * 8 + rr;
                const floatx4 t = *(const ASTERIA_LDS floatx4 *)(ws + r * 128 + ((e8 ^ (r & 7)) * 16));
                const size_t at = (size_t)(br + r) * P.ldc32 + bc;
                if (bf16) {
                    uint16_t *c = reinterpret_cast<uint16_t *>(P.C32) + at;
                    const uint32_t w0 = pg_pack_bf16(t[0], t[1]), w1 = pg_pack_bf16(t[2], t[3]);
                    if (vec) *(ASTERIA_GLOBAL u32x2_t *)c = (u32x2_t){w0, w1};
                    else { c[0] = (uint16_t)w0; c[1] = (uint16_t)(w0 >> 16); c[2] = (uint16_t)w1; c[3] = (uint16_t)(w1 >> 16); }
                } else {
                    float *c = P.C32 + at;
                    if (vec) *(ASTERIA_GLOBAL floatx4 *)c = t;
                    else { c[0] = t[0]; c[1] = t[1]; c[2] = t[2]; c[3] = t[3]; }
                }
            }
        }
}

template <int NTB, bool F16 = false>
__global__ __launch_bounds__(2 * PG_TILE, 2) void pgemm_kernel(const PlaneProblem *__restrict__ probs, int nprobs, int total_tiles)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int per_xcd = (total_tiles + NUM_XCD - 1) / NUM_XCD;
    const int t_global = (int)(blockIdx.x % NUM_XCD) * per_xcd + (int)(blockIdx.x / NUM_XCD);
    if (t_global >= total_tiles) return;
    pgemm_tile<NTB, F16, PG_TILE>(probs, nprobs, t_global, smem_raw);
}

// a plain fp32 matrix can feed pgemm_kernel: 16-byte aligned rows, whole tiles and slabs
inline bool pg_f32_operand_ok(const void *p, int rows, int k, int ld, int tile = PG_TILE)
{
    return (reinterpret_cast<uintptr_t>(p) & 15u) == 0 && (ld % 4) == 0 && (rows % tile) == 0 &&
           (k % PG_BK) == 0;
}

// a bf16 matrix can be B of pgemm_kernel<1>
inline bool pg_bf16_operand_ok(const void *p, int rows, int k, int ld)
{
    return (reinterpret_cast<uintptr_t>(p) & 15u) == 0 && (ld % 8) == 0 && (rows % PG_TILE) == 0 &&
           (k % PG_BK) == 0;
}

// Whether the whole-tile blocks of a call run on 256 x 256 tiles (one workgroup per CU, 256 at a time) or on
// the 128 x 128 ones of gemm_bf16.h (four times as many, 512 at a time); `tiles`: 256 x 256 tiles of the call,
// `tiles_k`: their sum of K.  A round of 512 small tiles takes 0.7 of a round of 256 large ones, so small ones pay only while
// they fit one round, 128 large tiles; at K = 256 the wide stores of the large tiles' epilogue count for more.  Time on small
// over large tiles, precondition (fp32 out) and soap_step: K = 1024, 64 tiles 0.71 0.69, 128: 0.87 0.88, 160: 1.25 1.24,
// 256: 1.43 1.32, 288: 0.99 1.03, 384: 1.14 1.15, 1024: 1.33 1.29; K = 2048, 128: 0.86 0.85, 192: 1.30 1.33, 320: 1.03 1.06;
// K = 512, 96: 0.98 0.96, 128: 1.00 0.99, 192: 1.32 1.30; K = 256, 32: 0.94 0.89, 64: 1.10 1.03, 128: 1.36 1.24.
inline bool pg_take_large_tiles(long long tiles, long long tiles_k)
{
    return tiles > (tiles_k < 512 * tiles ? 48 : 128);
}

template <int NTB, bool F16 = false>
inline hipError_t launch_pgemm(const PlaneProblem *probs, int nprobs, int total_tiles, hipStream_t stream, int kind)
{
    if (total_tiles <= 0 || nprobs <= 0) return hipSuccess;
    auto kern = pgemm_kernel<NTB, F16>;
    constexpr size_t lds = pg_lds_bytes(NTB, PG_TILE);
    static bool configured[MAX_DEVICES] = {};
    if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kern), lds, configured); e != hipSuccess) return e;
    const int per_xcd = (total_tiles + NUM_XCD - 1) / NUM_XCD;
    profile_begin(kind, stream);
    hipLaunchKernelGGL(kern, dim3(per_xcd * NUM_XCD), dim3(2 * PG_TILE), lds, stream, probs, nprobs, total_tiles);
    profile_end(stream);
    return hipGetLastError();
}

}  // namespace asteria
