// The orthonormalisation of one 128-row panel in the eigenbasis refresh: Gram matrix (fp64), Cholesky factor
// and its inverse (fp64), application of the inverse to the panel (fp32), which also leaves the finished rows
// as columns of the caller's Q.  The three kernels run once per sweep and panel, for all factors of a group.
#pragma once
#include <type_traits>

#include "gemm.h"

namespace asteria {

constexpr int QR_PANEL = 128;

// Orthonormalisation of Z^T (row c of Zt = column c of Z), in place.
struct QrFactor {
    float *Zt;      // n x ldz; rows become the orthonormal columns of Q, in order
    float *Qout;    // caller's Q (n x ldq)
    double *gram;   // partial Gram matrices of the current panel, see panel_gram_kernel
    float *winv;    // QR_PANEL x QR_PANEL: inverse Cholesky factor of the current panel, see panel_chol_kernel
    int n, ldz, ldq;
    int pad0_;
    int bad;        // set to 1 when a column could not be normalised
    // Two words the grouped launches read as their per-problem state (a problem runs while its word
    // is 0): `run` stays 0; `skip3` is 1 unless the second sweep over the current panel found a row
    // that needs a third one.
    int run, skip3;
    int out_index;  // position of this factor in the caller's arrays
    int pad_;
    // Powers of two that bring the rows of the current panel into the fp16 range for the projection
    // coefficients computed on the fp16 cores: a_scale for rows of Z^T as they come out of Q^T A
    // (bounded by tr A), 2^14 once a sweep has normalised them; p_scale is the one in force.
    float a_scale, p_scale;
    const float *A;  // the statistic (read for its trace)
    int lda, pad2_;
    float *cbuf;     // QR_PANEL rows x ldz for each panel in work: projection coefficients (gram and winv lie over them)
    // Where Q^T stands when a round starts (rows q_i^T: the k-contiguous operand of Z^T = Q^T A): the
    // caller's Q buffer, transposed in place, or a buffer of the caller that holds Q^T beside Q
    float *Qt;
    int ldqt, pad3_;
    double *est;     // n estimated eigenvalues q_i^T A q_i (column order of the refresh's input)
    int *perm;       // n: perm[r] = input column that becomes column r
    int *perm_out;   // the caller's slice of the permutation output, or null
};
constexpr float QR_UNIT_SCALE = 16384.0f;

// ---- Gram matrix ---------------------------------------------------------------------------------------
// G = P P^T of the panel's rows, fp64 products and sums, as 36 blocks of 16 x 16 on and below the diagonal.
// Wavefront w holds block rows 7 - w and w (9 blocks); in both operands of v_mfma_f64_16x16x4 lane i + 16 k
// holds element (i, k), so one register per block row and k serves as either, and operands come straight from
// memory (32 consecutive k of 16 rows, the four wavefronts share them in L1).
// A workgroup sums one of gram_splits(n) ranges of k - by n alone, so that a factor's result does not depend
// on what it is batched with - and stores its blocks in register order; panel_chol_kernel adds the ranges.
// Bound by the fp64 matrix cores (126 us for 260 factors of n = 2048).
constexpr int GRAM_BLOCKS = 36;
constexpr int GRAM_MAX_SPLITS = 6;
__host__ __device__ inline int gram_splits(int n)
{
    const int s = (n + 191) / 192;
    return s < GRAM_MAX_SPLITS ? s : GRAM_MAX_SPLITS;
}
__host__ __device__ inline size_t gram_doubles(int n) { return (size_t)gram_splits(n) * GRAM_BLOCKS * 256; }

template <int W>
__device__ __forceinline__ void gram_wave(const float *P, int ldz, int rows, int n, int k0, int k1, int lane, double *out)
{
    constexpr int NB = 8 - W;                        // block rows 0 .. 7 - W are operands
    const int r = lane & 15, h = lane >> 4;
    const ASTERIA_GLOBAL float *p[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) p[b] = (const ASTERIA_GLOBAL float *)(P + (size_t)min(16 * b + r, rows - 1) * ldz);
    doublex4 acc[9];
#pragma unroll
    for (int s = 0; s < 9; ++s)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[s][v] = 0.0;
    floatx4 cur[NB][2], nxt[NB][2];
    // lane group h takes k + 8 h .. k + 8 h + 7: any assignment of k to lanes and steps gives the same sum
    auto load = [&](floatx4 (&dst)[NB][2], int k) {
        const int kk = k + 8 * h;
        if (k + 32 <= n) {
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                dst[b][0] = *(const ASTERIA_GLOBAL floatx4 *)(p[b] + kk);
                dst[b][1] = *(const ASTERIA_GLOBAL floatx4 *)(p[b] + kk + 4);
            }
        } else {
            // rows are padded to whole groups of 4; what lies beyond n is not data
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int k4 = kk + 4 * q;
                    floatx4 t = {0.0f, 0.0f, 0.0f, 0.0f};
                    if (k4 < n) t = *(const ASTERIA_GLOBAL floatx4 *)(p[b] + k4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) dst[b][q][e] = k4 + e < n ? t[e] : 0.0f;
                }
        }
    };
    load(cur, k0);
    for (int k = k0; k < k1; k += 32) {
        if (k + 32 < k1) load(nxt, k + 32);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            double d[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) d[b] = (double)cur[b][e >> 2][e & 3];
#pragma unroll
            for (int j = 0; j < NB; ++j) acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(d[NB - 1], d[j], acc[j], 0, 0, 0);
#pragma unroll
            for (int j = 0; j <= W; ++j) acc[NB + j] = __builtin_amdgcn_mfma_f64_16x16x4f64(d[W], d[j], acc[NB + j], 0, 0, 0);
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) { cur[b][0] = nxt[b][0]; cur[b][1] = nxt[b][1]; }
    }
#pragma unroll
    for (int s = 0; s < 9; ++s) *(ASTERIA_GLOBAL doublex4 *)(out + ((size_t)(W * 9 + s) * 64 + lane) * 4) = acc[s];
}

__global__ __launch_bounds__(256, 2) void panel_gram_kernel(const QrFactor *__restrict__ fs, int panel, int sweep)
{
    const QrFactor &F = fs[blockIdx.y];              // the factors that have this panel are the first ones (sorted by size)
    if (sweep == 2 && F.skip3) return;
    const int splits = gram_splits(F.n), part = (int)blockIdx.x;
    if (part >= splits) return;
    const int chunk = ((F.n + splits - 1) / splits + 31) / 32 * 32;
    const int k0 = part * chunk, k1 = min(F.n, k0 + chunk);
    const int rows = min(QR_PANEL, F.n - panel * QR_PANEL);
    const float *P = F.Zt + (size_t)panel * QR_PANEL * F.ldz;
    double *out = F.gram + (size_t)part * GRAM_BLOCKS * 256;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // an empty last range stores zeros
    if (wave == 0) gram_wave<0>(P, F.ldz, rows, F.n, min(k0, F.n), k1, lane, out);
    else if (wave == 1) gram_wave<1>(P, F.ldz, rows, F.n, min(k0, F.n), k1, lane, out);
    else if (wave == 2) gram_wave<2>(P, F.ldz, rows, F.n, min(k0, F.n), k1, lane, out);
    else gram_wave<3>(P, F.ldz, rows, F.n, min(k0, F.n), k1, lane, out);
}

// ---- Cholesky factor and its inverse ---------------------------------------------------------------------
// One workgroup per (factor, panel).  In: the Gram matrix G = P P^T.  Out: W = L^-1 in fp32, where G = L L^T
// with a positive diagonal, so that W P has orthonormal rows and P = L (W P) is the QR relation with a positive
// diagonal.  All arithmetic in fp64.
//
// A pivot that is not positive (a zero row cannot be normalised) fails the factor.  In the second sweep over a
// panel (sweep = 1) the rows are those the first sweep normalised, projected once more: a pivot far below 1
// there means that a row was numerically dependent - the first normalisation blew round-off up to unit length,
// most of which lay in the span of the rows before it - and this sweep's normalisation amplifies what the
// projection left by 1 / sqrt(pivot).  Such a factor takes a third sweep (skip3 = 0), which only its workgroups
// run; a pivot that small in the third sweep fails the factor.
//
// The time is a chain of 128 pivots, so everything is laid out to keep a link short.  Eliminating column k acts
// in the same way on a row of A below it (it becomes a row of L), on a row of the diagonal block, and on a column
// of the identity (it becomes a column of W): v_k *= 1 / L_kk, v_i -= v_k L_ik.  So a block column of 16 takes
// one pass in registers, lane = row or column, multipliers from the lanes of the diagonal block (readlane), each
// of the four wavefronts with its own copy of that block - no barrier inside.  What remains, A and W to the right
// and below, lives in MFMA accumulators (block rows 7 - w and w of the lower triangle in wavefront w; block
// (i, j) is A for j > kb and W for j <= kb) and takes one rank-16 update per block column.
// One panel: 190 us before (LDS, serial inner loops), 36 now.
constexpr double CHOL_REPEAT_MIN = 0.1;
constexpr int CHOL_NB = 16;
constexpr int CHOL_PITCH = CHOL_NB + 2;              // doubles; rows stay 16-byte aligned
constexpr int CHOL_BLOCK = CHOL_NB * CHOL_PITCH;

__device__ __forceinline__ double lane_value(double v, int lane)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// 1 / sqrt(x) for positive normal x: one step of the third-order iteration from the hardware's estimate (measured: 5.2e-8 of relative
// error before it, 1.4e-16 after it and after a second one)
__device__ __forceinline__ double inv_sqrt(double x)
{
    const double y = __builtin_amdgcn_rsq(x), e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// where element (row, k) of W lies: the order in which the lanes of panel_apply_kernel read it
__device__ __forceinline__ int winv_off(int row, int k)
{
    return (((row >> 5) * 16 + (k >> 3)) * 64 + (row & 31) + 32 * ((k >> 2) & 1)) * 4 + (k & 3);
}

__global__ __launch_bounds__(256, 2) void panel_chol_kernel(QrFactor *fs, int panel, int sweep)
{
    QrFactor &F = fs[blockIdx.x];
    if (sweep == 2 && F.skip3) return;               // uniform over the workgroup
    const int rows = min(QR_PANEL, F.n - panel * QR_PANEL), nblk = (rows + CHOL_NB - 1) / CHOL_NB;
    __shared__ __align__(16) double in_[8 * CHOL_BLOCK], out_[8 * CHOL_BLOCK];
    __shared__ int bad_flag;
    ASTERIA_LDS double *in = (ASTERIA_LDS double *)in_, *pb = (ASTERIA_LDS double *)out_;
    typedef double dx2 __attribute__((ext_vector_type(2)));
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, h = lane >> 4;
    if (tid == 0) bad_flag = 0;
    doublex4 acc[2][8];                              // block rows i = 7 - w and w; [1][4 .. 7] unused
    {
        const int splits = gram_splits(F.n);
        const ASTERIA_GLOBAL double *g = (const ASTERIA_GLOBAL double *)F.gram;
        // The loads of a range stand side by side, blocks beyond the diagonal included (a copy of the last one): a branch around each
        // block waits for each, nine times a memory latency
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int j = 0; j < (q == 0 ? 8 : 4); ++j) acc[q][j] = (doublex4){0.0, 0.0, 0.0, 0.0};
        for (int s = 0; s < splits; ++s) {
            doublex4 t[12];
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int j = 0; j < (q == 0 ? 8 : 4); ++j) {
                    const int i = q == 0 ? 7 - w : w, slot = (q == 0 ? 9 * w : 9 * w + 8 - w) + min(j, i);
                    t[8 * q + j] = *(const ASTERIA_GLOBAL doublex4 *)(g + ((size_t)(s * GRAM_BLOCKS + slot) * 64 + lane) * 4);
                }
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int j = 0; j < (q == 0 ? 8 : 4); ++j) acc[q][j] += t[8 * q + j];
        }
        // rows and columns beyond `rows` are those of the identity: the blocks need no edge cases
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int j = 0; j < (q == 0 ? 8 : 4); ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int row = 16 * (q == 0 ? 7 - w : w) + 4 * v + h, col = 16 * j + r;
                    if (row >= rows || col >= rows) acc[q][j][v] = row == col ? 1.0 : 0.0;
                }
    }
    // block column kb (rows below) and the finished columns of block row kb, one vector of 16 per lane of the pass
    auto hand_out = [&](int kb) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int i = q == 0 ? 7 - w : w;
#pragma unroll
            for (int j = 0; j < (q == 0 ? 8 : 4); ++j) {
                if (j > i) continue;
                if (j == kb) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) in[i * CHOL_BLOCK + (4 * v + h) * CHOL_PITCH + r] = acc[q][j][v];
                } else if (i == kb && j < kb) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) in[j * CHOL_BLOCK + r * CHOL_PITCH + 4 * v + h] = acc[q][j][v];
                }
            }
        }
    };
    hand_out(0);
    __syncthreads();
    for (int kb = 0; kb < nblk; ++kb) {
        // lanes 0 .. 15: the diagonal block; 16 .. 47: this wavefront's two blocks; 48 .. 63: copies
        const int b = h == 0 ? kb : min(2 * w + h - 1, 2 * w + 1);
        double v[CHOL_NB];
        {
            const ASTERIA_LDS double *src = in + b * CHOL_BLOCK + r * CHOL_PITCH;
#pragma unroll
            for (int k = 0; k < CHOL_NB; k += 2) {
                const dx2 t = *(const ASTERIA_LDS dx2 *)(src + k);
                v[k] = t[0]; v[k + 1] = t[1];
            }
        }
        if (h != 0 && b == kb) {                     // columns of the identity
#pragma unroll
            for (int k = 0; k < CHOL_NB; ++k) v[k] = k == r ? 1.0 : 0.0;
        }
        int bad = 0;
        double low = 1.0;
        auto scale_of = [&](int k) __attribute__((always_inline)) {
            double piv = lane_value(v[k], k);
            if (!(piv > 0.0) || !(piv < 1e300)) {            // not positive definite: keep going with a tiny pivot
                bad = 1;
                piv = 1e-300;
            }
            low = fmin(low, piv);
            return inv_sqrt(piv);
        };
        double rd = scale_of(0);
#pragma unroll
        for (int k = 0; k < CHOL_NB; ++k) {
            const double t = v[k] * rd;
            v[k] = t;
            if (k + 1 < CHOL_NB) {
                // the next pivot first: its square root runs beside the other updates
                v[k + 1] = fma(-t, lane_value(t, k + 1), v[k + 1]);
                rd = scale_of(k + 1);
                // (four multipliers at a time: a scalar can be used two instructions after it was fetched)
#pragma unroll
                for (int i0 = k + 2; i0 < CHOL_NB; i0 += 4) {
                    double m[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) if (i0 + e < CHOL_NB) m[e] = lane_value(t, i0 + e);
#pragma unroll
                    for (int e = 0; e < 4; ++e) if (i0 + e < CHOL_NB) v[i0 + e] = fma(-t, m[e], v[i0 + e]);
                }
                // without this the multipliers of several columns are fetched ahead and spill
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (bad == 0 && sweep > 0 && low < CHOL_REPEAT_MIN) bad = 2;
        if (bad && tid == 0 && bad_flag != 1) bad_flag = bad;
        if (h == 1 || h == 2) {
            ASTERIA_LDS double *dst = pb + b * CHOL_BLOCK + r * CHOL_PITCH;
#pragma unroll
            for (int k = 0; k < CHOL_NB; k += 2) *(ASTERIA_LDS dx2 *)(dst + k) = (dx2){v[k], v[k + 1]};
            const bool zero = b == kb + 1 && (kb & 1) == 0;  // above the diagonal, inside a 32 x 32 block that is read
            if (b <= kb || zero) {
                ASTERIA_GLOBAL float *wo = (ASTERIA_GLOBAL float *)F.winv;
#pragma unroll
                for (int k = 0; k < CHOL_NB; ++k) wo[winv_off(16 * kb + k, 16 * b + r)] = zero ? 0.0f : (float)v[k];
            }
        }
        __syncthreads();
        // (i, j) -= (i, kb) (kb, j) for i > kb
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int i = q == 0 ? 7 - w : w;
            if (i <= kb || i >= nblk) continue;
            dx2 a[2];
            const ASTERIA_LDS double *pa = pb + i * CHOL_BLOCK + r * CHOL_PITCH + 4 * h;
            a[0] = *(const ASTERIA_LDS dx2 *)pa; a[1] = *(const ASTERIA_LDS dx2 *)(pa + 2);
            dx2 bb[8][2];
#pragma unroll
            for (int j = 0; j < (q == 0 ? 8 : 4); ++j) {
                const ASTERIA_LDS double *pj = pb + min(j, i) * CHOL_BLOCK + r * CHOL_PITCH + 4 * h;
                bb[j][0] = *(const ASTERIA_LDS dx2 *)pj; bb[j][1] = *(const ASTERIA_LDS dx2 *)(pj + 2);
            }
#pragma unroll
            for (int j = 0; j < (q == 0 ? 8 : 4); ++j) {
                if (j > i) continue;
                if (j == kb) acc[q][j] = (doublex4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    acc[q][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[e >> 1][e & 1], bb[j][e >> 1][e & 1], acc[q][j], 0, 0, 0);
            }
        }
        if (kb + 1 < nblk) hand_out(kb + 1);
        __syncthreads();
    }
    if (tid == 0) {
        if (bad_flag == 1 || (bad_flag == 2 && sweep == 2)) F.bad = 1;
        if (sweep == 0) { F.skip3 = 1; F.p_scale = QR_UNIT_SCALE; }       // the rows are normalised now
        // after the last sweep of a panel the scale goes back to that of the rows of Z^T (the next panel)
        if (sweep == 1) { if (bad_flag == 2) F.skip3 = 0; else F.p_scale = F.a_scale; }
        if (sweep == 2) F.p_scale = F.a_scale;
    }
}

// ---- P <- W P ----------------------------------------------------------------------------------------------
// One wavefront per 32 columns of a panel, fp32 matrix cores: the strip (64 registers) and the 10 blocks of 32 x 32
// on and below the diagonal of W, whose operands arrive in the order the Cholesky kernel left them, no LDS.  After
// the panel's last sweep the strip also goes to the caller's Q as columns and to a kept Q^T as rows.
// Bound by memory (the panel in and out).
__global__ __launch_bounds__(256, 2) void panel_apply_kernel(const QrFactor *__restrict__ fs, int panel, int sweep)
{
    const QrFactor &F = fs[blockIdx.y];
    if (sweep == 2 && F.skip3) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 31, h = lane >> 5;
    const int n = F.n, done = panel * QR_PANEL, rows = min(QR_PANEL, n - done);
    const int c0 = ((int)blockIdx.x * 4 + wave) * 32;
    if (c0 >= n) return;
    const bool final = sweep == 2 || (sweep == 1 && F.skip3);
    const int col = c0 + r, cc = min(col, n - 1), ldz = F.ldz;
    ASTERIA_GLOBAL float *P = (ASTERIA_GLOBAL float *)(F.Zt + (size_t)done * ldz);
    const ASTERIA_GLOBAL floatx4 *Wf = (const ASTERIA_GLOBAL floatx4 *)F.winv + lane;
    float x[16][4];
#pragma unroll
    for (int t = 0; t < 16; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int k = 8 * t + 4 * h + e;
            const float v = P[(uint32_t)min(k, rows - 1) * (uint32_t)ldz + (uint32_t)cc];   // 128 n 4 bytes fit 32 bits
            x[t][e] = k < rows ? v : 0.0f;
        }
    floatx16 acc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = 0.0f;
#pragma unroll
    for (int t = 0; t < 16; ++t) {
        floatx4 a[4];
#pragma unroll
        for (int i = t / 4; i < 4; ++i) a[i] = Wf[(i * 16 + t) * 64];
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = t / 4; i < 4; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][e], x[t][e], acc[i], 0, 0, 0);
    }
    if (col >= n) return;
    auto store = [&](auto whole) __attribute__((always_inline)) {
        constexpr bool WHOLE = decltype(whole)::value;           // all 128 rows are there
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = 32 * i + 8 * (v >> 2) + 4 * h + (v & 3);
                if (WHOLE || row < rows) P[(uint32_t)row * (uint32_t)ldz + (uint32_t)col] = acc[i][v];
            }
        if (!final) return;
        ASTERIA_GLOBAL float *Q = (ASTERIA_GLOBAL float *)(F.Qout + (size_t)col * F.ldq + done);
        const bool vec = ((reinterpret_cast<uintptr_t>(F.Qout) & 15u) == 0) && ((F.ldq & 3) == 0);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int row = 32 * i + 8 * g + 4 * h;
                if (vec && (WHOLE || row + 4 <= rows)) {
                    *(ASTERIA_GLOBAL floatx4 *)(Q + row) = (floatx4){acc[i][4 * g], acc[i][4 * g + 1], acc[i][4 * g + 2], acc[i][4 * g + 3]};
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (WHOLE || row + e < rows) Q[row + e] = acc[i][4 * g + e];
                }
            }
        if (F.Qt != F.Qout) {
            ASTERIA_GLOBAL float *T = (ASTERIA_GLOBAL float *)(F.Qt + (size_t)done * F.ldqt + col);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = 32 * i + 8 * (v >> 2) + 4 * h + (v & 3);
                    if (WHOLE || row < rows) T[(size_t)row * F.ldqt] = acc[i][v];
                }
        }
    };
    if (rows == QR_PANEL) store(std::true_type{});
    else store(std::false_type{});
}

}  // namespace asteria
