// asteria_inverse_root: X = ((A + A^T)/2 + eps I)^(-1/p) for a batch of symmetric factors
// (the inverse roots of paper Eq. 1; the O(d^3) update of paper Sec. I / III-B), computed
// entirely on the device:
//
//   1. lambda_max(A) by a Lanczos process (HBM-streaming mat-vec, wavefront reductions, the small
//      tridiagonal eigenproblem per factor on the device, per-factor early stop).
//   2. Scaling  s = 1 / ((1 + margin) lambda_max + eps),  M_0 = s (A + eps I),  X_0 = s^(1/p) I,
//      so the spectrum of M_0 lies in (0, 1].
//   3. Coupled iteration  T = a I - g M,  X <- X T,  M <- T^p M  (coefficients a, g adapted per
//      factor and iteration to the interval that holds M's spectrum, or the classical Newton
//      values a = (p + 1) / p, g = 1 / p).  Every product is one symmetric grouped GEMM on the
//      matrix cores; the epilogue of the M-update also emits the next T and the per-tile partial
//      sums of ||M - I||_F^2.  A per-factor state machine on the device (running -> last X
//      update -> done) lets finished factors drop out without any host round trip: their
//      workgroups exit at once.
//   4. The leading iterations of the M-chain keep fp64 matrices, where the smallest eigenvalues
//      of M are still comparable to fp32 round-off.  Their products run on the int8 matrix cores:
//      each operand is cut into its diagonal and 7-bit integer slices under a per-row exponent,
//      the integer sums are exact and the result is assembled in fp64 (gemm_i8.h); per factor
//      and product a device-side estimate of what the dropped slice pairs cost picks 4 or 5
//      slices or sends the product to the fp64 matrix cores.  The state is then cast to fp32 and
//      continues on
//      the fp16 matrix cores with every fp32 operand split into two fp16 terms (2^-22 per
//      operand; the fp32 matrix cores serve pinned options, absolute eps and very large n).  X
//      is kept in fp32 throughout and its updates run on the fp16 cores from the start.
//
// Per iteration: 1 control kernel + up to 4 launches (X T; T T; T^2 T^2; T^4 M); in the fp64
// iterations each chain product is a slicing pass, a decision kernel, the int8 launch and the
// fp64 launch for the factors the decision kept there.
#include <math.h>
#include <stddef.h>

#include <algorithm>
#include <vector>

#include "common.h"
#include "gemm.h"
#include "gemm_bf16.h"
#include "gemm_i8.h"
#include "root_factor.h"
#include "root_lanczos.h"
#include "root_products.h"
#include "root_schedule.h"

using namespace asteria;

namespace {

// spectrum of M within 1 +- ROOT_STOP_DEV: one more X update finishes the factor
constexpr float ROOT_STOP_DEV = 1e-2f;
// accepted truncation error of the result per eigen-direction (a third of the 2e-3 accuracy bar
// on the relative Frobenius error, which averages over directions)
constexpr float ROOT_X_TOL = 7e-4f;

constexpr int PM_TILE_WORDS = 2 * PACK_T + 2;   // floats per tile in pm_tile: two vectors and a double

// Scale of M, T, T^2, T^4 in the fp16-split products: their entries stay below a^4 < 23 (a <= 2.2),
// so 2^10 keeps them under 2^15 with the fp16 range ending at 65504.
constexpr float ROOT_F16_SCALE = 1024.0f;

template <typename T> __device__ __forceinline__ T wave_sum(T v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// ---- lambda_max of large packed statistics (root_lanczos.h has the process and the other kernels) ---------
// one workgroup (256 threads) per factor: the unit start vector
__global__ __launch_bounds__(256) void pm_init_kernel(const FactorDev *fd, FactorScal *fs)
{
    const int f = blockIdx.x;
    const FactorDev &F = fd[f];
    __shared__ float red[4];
    float s = 0.0f;
    for (int j = threadIdx.x; j < F.n; j += 256) {
        // the same start vector for every factor: a factor's result does not depend on its place in the batch
        const float v = hash_unit(0u, (uint32_t)j);
        F.pv[0][j] = v;
        s += v * v;
    }
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    const float t = red[0] + red[1] + red[2] + red[3], inv = t > 0.0f ? rsqrtf(t) : 0.0f;
    for (int j = threadIdx.x; j < F.n; j += 256) F.pv[0][j] *= inv;      // the entries this thread has written
    if (threadIdx.x == 0) {
        fs[f].rho = 0.0f;
        fs[f].lz_small = 0;
        fs[f].pm_done = 0;
    }
}

// y = A v for LZ_ROWS rows of one factor in full storage, for batches that mix both storages and for factors
// whose vectors do not fit LDS.
__global__ __launch_bounds__(256) void pm_matvec_kernel(const FactorDev *fd, const FactorScal *fs, int src, int dst, int first)
{
    const int f = blockIdx.y;
    if (fs[f].pm_done) return;
    const FactorDev &F = fd[f];
    const int blk = (int)blockIdx.x;
    if (F.a_packed || blk >= F.pm_blocks) return;
    const int n = F.n;
    const float *__restrict__ v = F.pv[src];
    float *__restrict__ y = F.pv[dst];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __shared__ float red[4];
    __shared__ double redd[2][4];
    float syv = 0.0f;
    double saa = 0.0, str = 0.0;                      // saa: every lane its part
    for (int rr = 0; rr < LZ_ROWS / 4; ++rr) {
        const int row = blk * LZ_ROWS + wave * (LZ_ROWS / 4) + rr;
        if (row >= n) break;
        const float *__restrict__ a = F.A + (size_t)row * F.lda;
        float s = 0.0f;
#pragma unroll 4
        for (int j = lane; j < n; j += 64) { s += a[j] * v[j]; if (first) saa += (double)a[j] * (double)a[j]; }
        s = wave_sum(s);
        if (lane == 0) {
            y[row] = s;
            syv += s * v[row];
            str += (double)a[row];
        }
    }
    if (first) saa = wave_sum(saa);
    if (lane == 0) { red[wave] = syv; redd[0][wave] = saa; redd[1][wave] = str; }
    __syncthreads();
    if (threadIdx.x == 0) {
        F.pm_partial[blk] = red[0] + red[1] + red[2] + red[3];
        if (first)
            F.pm_partial2[blk] = make_double2(redd[0][0] + redd[0][1] + redd[0][2] + redd[0][3], redd[1][0] + redd[1][1] + redd[1][2] + redd[1][3]);
    }
}

// y = A v for statistics in packed lower tiles.
// One workgroup per stored tile (ti, tj), tj <= ti: it serves both the rows of block ti (T v_tj) and,
// off the diagonal, the rows of block tj (T^T v_ti), so every element is read once.  The partial
// products go to the factor's pm_tile array and are summed in a fixed order by pm_packed_reduce_kernel
// (no atomics: the result does not depend on the order in which workgroups finish).
__global__ __launch_bounds__(256) void pm_packed_tile_kernel(const FactorDev *fd, const FactorScal *fs, int src, int first)
{
    const int f = blockIdx.y;
    if (fs[f].pm_done) return;
    const FactorDev &F = fd[f];
    if (!F.a_packed || (int)blockIdx.x >= F.ntri) return;
    int ti, tj;
    tri_decode((int)blockIdx.x, ti, tj);
    const int n = F.n;
    const float *__restrict__ tile = F.A + (size_t)blockIdx.x * PACK_T * PACK_T;
    const float *__restrict__ v = F.pv[src];
    float *out = F.pm_tile + (size_t)blockIdx.x * PM_TILE_WORDS;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c0 = tj * PACK_T + 2 * lane, r0 = ti * PACK_T;
    __shared__ float colp[4][PACK_T];
    __shared__ double redd[4];
    // this lane's two columns of the tile: entries of v_tj, zero beyond n
    const float vj0 = c0 < n ? v[c0] : 0.0f, vj1 = c0 + 1 < n ? v[c0 + 1] : 0.0f;
    float cs0 = 0.0f, cs1 = 0.0f;
    double saa = 0.0;
    for (int rr = 0; rr < PACK_T / 4; ++rr) {
        const int r = wave * (PACK_T / 4) + rr, gr = r0 + r;
        float2 a = *reinterpret_cast<const float2 *>(tile + (size_t)r * PACK_T + 2 * lane);
        if (gr >= n) { a.x = 0.0f; a.y = 0.0f; }               // padding of a ragged last tile row is undefined
        if (c0 >= n) a.x = 0.0f;
        if (c0 + 1 >= n) a.y = 0.0f;
        float s = wave_sum(a.x * vj0 + a.y * vj1);
        if (lane == 0) out[r] = s;                              // row part: (T v_tj)[r]
        const float vi = gr < n ? v[gr] : 0.0f;
        cs0 += a.x * vi; cs1 += a.y * vi;                       // column part: (T^T v_ti)[c]
        if (first) saa += (double)a.x * (double)a.x + (double)a.y * (double)a.y;
    }
    colp[wave][2 * lane] = cs0; colp[wave][2 * lane + 1] = cs1;
    if (first) {
        saa = wave_sum(saa);
        if (lane == 0) redd[wave] = saa;
    }
    __syncthreads();
    if (threadIdx.x < PACK_T)
        out[PACK_T + threadIdx.x] = colp[0][threadIdx.x] + colp[1][threadIdx.x] + colp[2][threadIdx.x] + colp[3][threadIdx.x];
    if (first && threadIdx.x == 0) {
        // an off-diagonal tile stands for its mirror image too
        const double w = ti == tj ? 1.0 : 2.0;
        *reinterpret_cast<double *>(out + 2 * PACK_T) = w * (redd[0] + redd[1] + redd[2] + redd[3]);
    }
}

// y[rows of block I] = sum over tj <= I of the row parts of tile (I, tj) + sum over ti > I of the column
// parts of tile (ti, I); per block the same partial sums pm_matvec_kernel leaves.
__global__ __launch_bounds__(PACK_T) void pm_packed_reduce_kernel(const FactorDev *fd, const FactorScal *fs, int src, int dst, int first)
{
    const int f = blockIdx.y;
    if (fs[f].pm_done) return;
    const FactorDev &F = fd[f];
    const int T = (F.n + PACK_T - 1) / PACK_T, I = (int)blockIdx.x;
    if (!F.a_packed || I >= T) return;
    const int i = threadIdx.x, row = I * PACK_T + i;
    const float *__restrict__ v = F.pv[src];
    float s = 0.0f;
    double saa = 0.0, str = 0.0;
    if (first && row < F.n) str = (double)F.A[packed_off(row, row)];
    for (int tj = 0; tj <= I; ++tj) {
        const float *p = F.pm_tile + (size_t)(I * (I + 1) / 2 + tj) * PM_TILE_WORDS;
        s += p[i];
        if (first && i == 0) saa += *reinterpret_cast<const double *>(p + 2 * PACK_T);
    }
    for (int ti = I + 1; ti < T; ++ti) s += F.pm_tile[(size_t)(ti * (ti + 1) / 2 + I) * PM_TILE_WORDS + PACK_T + i];
    float syv = 0.0f;
    if (row < F.n) {
        F.pv[dst][row] = s;
        syv = s * v[row];
    }
    __shared__ float red[PACK_T / 64];
    __shared__ double redt[PACK_T / 64];
    syv = wave_sum(syv);
    if (first) str = wave_sum(str);
    if ((i & 63) == 0) { red[i >> 6] = syv; redt[i >> 6] = str; }
    __syncthreads();
    if (i == 0) {
        F.pm_partial[I] = red[0] + red[1];
        // the off-diagonal tiles of the block rows below this one were counted there (weight 2)
        if (first) F.pm_partial2[I] = make_double2(saa, redt[0] + redt[1]);
    }
}

// One workgroup per factor, after the mat-vec of step `it` (y = A v in pv[dst], v in pv[src], the vector
// before it in pv[prev]): alpha, the next Lanczos vector (over y), beta, the estimate, the stop.
// A factor stops once three consecutive steps have raised the estimate by less than tol2 of it (or the
// recurrence ends: beta = 0, an invariant subspace, where the estimate is exact).
__global__ __launch_bounds__(256) void pm_lanczos_kernel(const FactorDev *fd, FactorScal *fs, float tol2, int it,
                                                         int src, int dst, int prev, int first, int last)
{
    const int f = blockIdx.x;
    FactorScal &S = fs[f];
    if (S.pm_done) return;
    const FactorDev &F = fd[f];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float beta_p = it > 0 ? S.lz_b[it - 1] : 0.0f;
    __shared__ double red[3][4];
    // sums the mat-vec workgroups left per block of rows, in a fixed order
    double yv = 0.0, aa = 0.0, tr = 0.0;
    for (int b = tid; b < F.pm_blocks; b += 256) {
        yv += (double)F.pm_partial[b];
        if (first) { const double2 q = F.pm_partial2[b]; aa += q.x; tr += q.y; }
    }
    auto block_sum3 = [&](double &x0, double &x1, double &x2) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            x0 += __shfl_xor(x0, off, 64); x1 += __shfl_xor(x1, off, 64); x2 += __shfl_xor(x2, off, 64);
        }
        __syncthreads();
        if (lane == 0) { red[0][wave] = x0; red[1][wave] = x1; red[2][wave] = x2; }
        __syncthreads();
        x0 = red[0][0] + red[0][1] + red[0][2] + red[0][3]; x1 = red[1][0] + red[1][1] + red[1][2] + red[1][3];
        x2 = red[2][0] + red[2][1] + red[2][2] + red[2][3];
    };
    block_sum3(yv, aa, tr);
    const float alpha = (float)yv;                    // v is a unit vector: alpha = v^T A v
    // w = y - alpha v - beta_{j-1} v_{j-1}, written over y
    const float *__restrict__ v = F.pv[src], *__restrict__ vp = F.pv[prev];
    float *__restrict__ w = F.pv[dst];
    double ww = 0.0, z1 = 0.0, z2 = 0.0;
    for (int i = tid; i < F.n; i += 256) {
        float x = w[i] - alpha * v[i];
        if (it > 0) x -= beta_p * vp[i];
        w[i] = x;
        ww += (double)x * (double)x;
    }
    block_sum3(ww, z1, z2);
    if (first && tid == 0) { S.fro2 = aa; S.trace = tr; }
    const float beta = (float)sqrt(ww);
    if (!(beta < 3.0e38f) || !(fabsf(alpha) < 3.0e38f)) {
        if (tid == 0) { S.rho = NAN; S.pm_done = 1; }
        return;
    }
    // unit vectors throughout: A times an unnormalised one would be of the size of A squared
    const float inv = beta > 0.0f ? 1.0f / beta : 0.0f;
    for (int i = tid; i < F.n; i += 256) w[i] *= inv;
    __shared__ __align__(16) float la[LZ_MAX], lb[LZ_MAX];
    if (tid < it) { la[tid] = S.lz_a[tid]; lb[tid] = S.lz_b[tid]; }
    if (tid == 0) { S.lz_a[it] = la[it] = alpha; S.lz_b[it] = lb[it] = beta; }
    __syncthreads();
    if (wave != 0) return;
    const bool stop = lanczos_advance(S, la, lb, it, beta, tol2);
    if (lane == 0 && (stop || last)) S.pm_done = 1;
}

// ---- scaling and start of the coupled iteration ---------------------------------------------
__global__ void root_setup_kernel(const FactorDev *fd, FactorScal *fs, int *state, int nf,
                                  int relative, float margin, int root, int adapted)
{
    const int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= nf) return;
    FactorScal &S = fs[f];
    const float lam = S.rho;
    S.lam = lam;
    S.iters = 0;
    S.xloc = 0;
    S.resid = 0.0f;
    const float eps = relative ? fd[f].eps_in * lam : fd[f].eps_in;
    S.eps = eps;
    const float denom = (1.0f + margin) * lam + eps;
    const bool ok = (lam == lam) && (lam >= 0.0f) && (lam < 3.0e38f) && (denom > 0.0f) && (denom < 3.0e38f);
    if (!ok) {
        S.scale = 0.0f;
        S.info = ASTERIA_INFO_NOT_PD;
        state[f] = ST_FAIL;
    } else {
        S.scale = 1.0f / denom;
        S.info = ASTERIA_INFO_OK;
        state[f] = ST_RUN;
    }
    // spectrum of M_0 = s (A + eps I): at most 1 by the scaling; at least eps s for a positive
    // semi-definite A (halved: round-off in the statistics may push eigenvalues slightly below 0)
    double lo = ok ? 0.5 * (double)eps / (double)denom : 1.0;
    if (!(lo > 1e-12)) lo = 1e-12;
    if (ok) {
        // ||M_0 - I||_F^2 = s^2 ||A + eps I||_F^2 - 2 s tr(A + eps I) + n bounds every |mu - 1|:
        // a well-conditioned factor gets a much tighter interval than [eps s, 1]
        const double sc = 1.0 / (double)denom, e = (double)eps, n = (double)fd[f].n;
        const double f2 = S.fro2 + 2.0 * e * S.trace + n * e * e;
        const double tr = S.trace + n * e;
        double r2 = sc * sc * f2 - 2.0 * sc * tr + n;
        r2 = r2 * (1.0 + 1e-3) + 1e-6 * n;           // slack for the fp32 sums
        if (r2 > 0.0 && r2 < 1.0) { const double l1 = 1.0 - sqrt(r2); if (l1 > lo) lo = l1; }
    }
    // Every iterate X_k = xs prod T_j has eigenvalues x with (x / xs)^root lambda = mu <= 2, lambda >= lo
    // an eigenvalue of M_0 and mu the matching one of M_k: |X_k| <= xs (2 / lo)^(1/root).  The
    // fp16-split products scale X by the largest power of two that keeps this bound below 30000.
    {
        const double xs = ok ? pow((double)S.scale, 1.0 / (double)root) : 1.0;
        const double bound = xs * pow(2.0 / lo, 1.0 / (double)root);
        int e = (int)floor(log2(30000.0 / bound));
        e = e < -60 ? -60 : (e > 60 ? 60 : e);
        S.x_scale = (float)ldexp(1.0, e);
    }
    double a, g;
    root_coefficients(lo, 1.0, root, adapted != 0, ROOT_THETA, a, g);
    S.lo = (float)lo; S.hi = 1.0f;
    S.ca = (float)a; S.cg = (float)g;
    S.coef_next[0] = (float)a; S.coef_next[1] = (float)g;
}

// 4 consecutive elements as 16-byte stores (the destination is 16-byte aligned)
__device__ __forceinline__ void store4(float *p, const float (&v)[4])
{
    *reinterpret_cast<float4 *>(p) = make_float4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ void store4(double *p, const double (&v)[4])
{
    reinterpret_cast<double2 *>(p)[0] = make_double2(v[0], v[1]);
    reinterpret_cast<double2 *>(p)[1] = make_double2(v[2], v[3]);
}

// One workgroup per lower-triangle 128 x 128 tile: M_0, T_0, X_0 and the residual partial sums.
template <typename TC>
__global__ __launch_bounds__(256) void root_init_kernel(const FactorDev *fd, const FactorScal *fs,
                                                        const int *state, int nf, int total_tiles,
                                                        int root)
{
    const int t_global = blockIdx.x;
    if (t_global >= total_tiles) return;
    int lo = 0, hi = nf - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (fd[mid].tile_start <= t_global) lo = mid; else hi = mid - 1;
    }
    const FactorDev &F = fd[lo];
    if (state[lo] != ST_RUN) return;
    const int lt = t_global - F.tile_start;
    int ti, tj;
    tri_decode(lt, ti, tj);
    const int n = F.n, lda = F.lda;
    const TC s = (TC)fs[lo].scale;
    const TC eps = (TC)fs[lo].eps;
    const TC xs = (TC)pow((double)fs[lo].scale, 1.0 / (double)root);
    const TC ca = (TC)fs[lo].ca, cg = (TC)fs[lo].cg;
    // X_0 = xs I is never stored: the first update X_1 = X_0 T_0 = xs T_0 is written directly
    // (into the buffer that holds X after an odd number of updates), which saves one product.
    TC *M, *T;
    int ldm;
    if (sizeof(TC) == 8) {
        M = reinterpret_cast<TC *>(F.M64[0]); T = reinterpret_cast<TC *>(F.T64); ldm = F.ld64;
    } else {
        M = reinterpret_cast<TC *>(F.M32[0]); T = reinterpret_cast<TC *>(F.T32); ldm = F.ld32;
    }
    float *X = F.X32b;            // holds X after an odd number of updates
    // no fp32 copy of T_0 is needed: X_1 = xs T_0 is written here, and the first X product (k = 1)
    // reads the fp32 T_1 that the M-update epilogue of iteration 0 writes
    const int ldx = F.ld32;
    // The tile pair (ti, tj) / (tj, ti) is walked in 32 x 32 sub-tiles.  P = A[sub(ti, tj)] and
    // Q = A[sub(tj, ti)] are both read along rows (coalesced) into LDS; the symmetrised value at
    // (r, c) of tile (ti, tj) is (P[r][c] + Q[c][r]) / 2 and the one at (c, r) of tile (tj, ti) is
    // the same number, so every global read and write of this kernel runs along rows.
    float rsum = 0.0f;
    __shared__ float red[4];
    // Full tiles with 16-byte aligned rows: 64 x 64 sub-tiles, 16-byte global loads, and 32-byte
    // (fp64) or 16-byte (fp32) stores of 4 consecutive elements per thread; LDS rows of 65 words
    // keep both the row-wise and the transposed reads free of bank conflicts.
    // Packed lower tiles: tile (ti, tj) is stored once, dense with 128 floats per row, and stands for
    // its mirror image; the value at (r, c) is the stored one (nothing to symmetrise).
    const bool packed = F.a_packed != 0;
    const float *Ap = packed ? F.A + (size_t)lt * PACK_T * PACK_T : nullptr;
    const bool aligned = ti * BM + BM <= n && (packed || ((lda & 3) == 0 && (reinterpret_cast<uintptr_t>(F.A) & 15u) == 0));
    if (aligned) {
        __shared__ float Pw[64][65], Qw[64][65];
        const int g = threadIdx.x & 15, rw = threadIdx.x >> 4;     // 16 column groups of 4 x 16 rows
        for (int sub = 0; sub < 4; ++sub) {
            const int si = sub >> 1, sj = sub & 1;
            if (ti == tj && si < sj) continue;                       // covered by the mirrored sub-tile
            const int r0 = ti * BM + si * 64, c0 = tj * BN + sj * 64;
            const bool diag_sub = (ti == tj && si == sj);
            __syncthreads();
            for (int rr = rw; rr < 64; rr += 16) {
                const float4 pv = packed ? *reinterpret_cast<const float4 *>(Ap + (size_t)(si * 64 + rr) * PACK_T + sj * 64 + 4 * g)
                                         : *reinterpret_cast<const float4 *>(F.A + (size_t)(r0 + rr) * lda + c0 + 4 * g);
                Pw[rr][4 * g] = pv.x; Pw[rr][4 * g + 1] = pv.y; Pw[rr][4 * g + 2] = pv.z; Pw[rr][4 * g + 3] = pv.w;
                if (!packed) {
                    const float4 qv = *reinterpret_cast<const float4 *>(F.A + (size_t)(c0 + rr) * lda + r0 + 4 * g);
                    Qw[rr][4 * g] = qv.x; Qw[rr][4 * g + 1] = qv.y; Qw[rr][4 * g + 2] = qv.z; Qw[rr][4 * g + 3] = qv.w;
                }
            }
            __syncthreads();
            for (int rr = rw; rr < 64; rr += 16) {
                // elements (r, c .. c + 3) of tile (ti, tj)
                {
                    const int r = r0 + rr, c = c0 + 4 * g;
                    TC mv[4], tv[4];
                    float xv[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const TC av = packed ? (TC)Pw[rr][4 * g + e] : (TC)0.5 * ((TC)Pw[rr][4 * g + e] + (TC)Qw[4 * g + e][rr]);
                        const TC d = (r == c + e) ? (TC)1 : (TC)0;
                        mv[e] = s * (av + eps * d);
                        tv[e] = ca * d - cg * mv[e];
                        xv[e] = (float)(xs * tv[e]);
                        const float er = (float)(mv[e] - d);
                        rsum += diag_sub ? er * er : 2.0f * er * er;
                    }
                    store4(M + (size_t)r * ldm + c, mv);
                    store4(T + (size_t)r * ldm + c, tv);
                    store4(X + (size_t)r * ldx + c, xv);
                }
                // elements (r2, c2 .. c2 + 3) of the mirrored tile (tj, ti): the same numbers transposed
                if (!diag_sub) {
                    const int r2 = c0 + rr, c2 = r0 + 4 * g;
                    TC mv[4], tv[4];
                    float xv[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const TC av = packed ? (TC)Pw[4 * g + e][rr] : (TC)0.5 * ((TC)Pw[4 * g + e][rr] + (TC)Qw[rr][4 * g + e]);
                        mv[e] = s * av;                              // off the diagonal: no eps, d = 0
                        tv[e] = -cg * mv[e];
                        xv[e] = (float)(xs * tv[e]);
                    }
                    store4(M + (size_t)r2 * ldm + c2, mv);
                    store4(T + (size_t)r2 * ldm + c2, tv);
                    store4(X + (size_t)r2 * ldx + c2, xv);
                }
            }
        }
        rsum = wave_sum(rsum);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = rsum;
        __syncthreads();
        if (threadIdx.x == 0) { F.partial[lt] = red[0] + red[1] + red[2] + red[3]; F.partial[F.ntri + lt] = 0.0f; }
        return;
    }
    __shared__ float Ps[32][33], Qs[32][33];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;     // 32 x 8 threads
    for (int sub = 0; sub < 16; ++sub) {
        const int si = sub >> 2, sj = sub & 3;
        const int r0 = ti * BM + si * 32, c0 = tj * BN + sj * 32;
        if (r0 >= n || c0 >= n) continue;                        // uniform over the workgroup
        if (ti == tj && si < sj) continue;                       // covered by the mirrored sub-tile
        __syncthreads();
        for (int rr = ty; rr < 32; rr += 8) {
            const int r = r0 + rr, c = c0 + tx;
            Ps[rr][tx] = (r < n && c < n) ? (packed ? Ap[(size_t)(si * 32 + rr) * PACK_T + sj * 32 + tx] : F.A[(size_t)r * lda + c]) : 0.0f;
            const int r2 = c0 + rr, c2 = r0 + tx;                // sub-tile (sj, si) of tile (tj, ti)
            if (!packed) Qs[rr][tx] = (r2 < n && c2 < n) ? F.A[(size_t)r2 * lda + c2] : 0.0f;
        }
        __syncthreads();
        const bool diag_sub = (ti == tj && si == sj);
        for (int rr = ty; rr < 32; rr += 8) {
            // element (r, c) of tile (ti, tj)
            {
                const int r = r0 + rr, c = c0 + tx;
                if (r < n && c < n) {
                    const TC av = packed ? (TC)Ps[rr][tx] : (TC)0.5 * ((TC)Ps[rr][tx] + (TC)Qs[tx][rr]);
                    const TC d = (r == c) ? (TC)1 : (TC)0;
                    const TC m = s * (av + eps * d);
                    const TC t = ca * d - cg * m;
                    M[(size_t)r * ldm + c] = m;
                    T[(size_t)r * ldm + c] = t;
                    X[(size_t)r * ldx + c] = (float)(xs * t);
                    const float e = (float)(m - d);
                    // a diagonal sub-tile holds both triangles itself; every other one stands for two
                    rsum += diag_sub ? e * e : 2.0f * e * e;
                }
            }
            // element (r2, c2) of the mirrored tile (tj, ti): same value, written along its own rows
            if (!diag_sub) {
                const int r2 = c0 + rr, c2 = r0 + tx;
                if (r2 < n && c2 < n) {
                    const TC av = packed ? (TC)Ps[tx][rr] : (TC)0.5 * ((TC)Ps[tx][rr] + (TC)Qs[rr][tx]);
                    const TC m = s * av;                          // off the diagonal: no eps, d = 0
                    const TC t = -cg * m;
                    M[(size_t)r2 * ldm + c2] = m;
                    T[(size_t)r2 * ldm + c2] = t;
                    X[(size_t)r2 * ldx + c2] = (float)(xs * t);
                }
            }
        }
    }
    rsum = wave_sum(rsum);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = rsum;
    __syncthreads();
    if (threadIdx.x == 0) { F.partial[lt] = red[0] + red[1] + red[2] + red[3]; F.partial[F.ntri + lt] = 0.0f; }
}

// One wavefront per factor, run before iteration k (and once after the last one with
// final_pass = 1): evaluates the residual of running factors and advances the state machine.
__global__ __launch_bounds__(64) void root_control_kernel(const FactorDev *fd, FactorScal *fs, int *state,
                                                          int k, int fp32_phase, int final_pass,
                                                          float stop_resid, int root, int adapted, int look_ahead)
{
    const int f = blockIdx.x;
    const FactorDev &F = fd[f];
    FactorScal &S = fs[f];
    int st = state[f];
    if (st == ST_DONE || st == ST_FAIL) return;
    if (st == ST_LAST) {
        st = ST_DONE;
    } else {
        float r2 = 0.0f;
        // the int8 product writes two partial sums per tile (one per half), the other kernels the
        // first only: the second is cleared once read
        for (int i = threadIdx.x; i < F.ntri; i += 64) {
            r2 += F.partial[i] + F.partial[F.ntri + i];
            F.partial[F.ntri + i] = 0.0f;
        }
        r2 = wave_sum(r2);
        const float resid = sqrtf(r2);
        if (!(r2 == r2) || !(r2 < 3.0e38f)) {
            st = ST_FAIL;
            if (threadIdx.x == 0) { S.info = ASTERIA_INFO_NOT_PD; S.resid = resid; }
        } else {
            if (threadIdx.x == 0) S.resid = resid;
            // Last X update now?  X_{k+1} = X_k T_k differs from the root by |mu - 1| / 4 per eigen-
            // direction, mu in the spectrum of M_{k+1}.  Three ways to know that this is small:
            //  - the measured residual of M_k is below stop_resid (the update squares it);
            //  - the interval predicted for M_k has contracted to 1 +- ROOT_STOP_DEV;
            //  - the image of that interval under this iteration's map, i.e. the interval of
            //    M_{k+1}, lies within 1 +- 4 ROOT_X_TOL: M_{k+1} need not be formed at all.
            // The predictions are trusted only while the measured residual is consistent with
            // them: every |mu - 1| is at most ||M_k - I||_F, so an eigenvalue far outside shows.
            const float dev = fmaxf(1.0f - S.lo, S.hi - 1.0f);
            const bool consistent = resid < 1.5f * sqrtf((float)F.n) * dev + 2e-3f;
            double lo_k = (double)S.lo, hi_k = (double)S.hi;
            const double rb = (double)resid * 1.001 + 1e-5;
            if (1.0 - rb > lo_k) lo_k = 1.0 - rb;
            if (1.0 + rb < hi_k) hi_k = 1.0 + rb;
            if (!(hi_k > lo_k)) { lo_k = 1.0 - rb; hi_k = 1.0 + rb; }
            const RootInterval nx = root_image(lo_k, hi_k, root, (double)S.ca, (double)S.cg);
            const double dev_next = fmax(1.0 - nx.lo, nx.hi - 1.0);
            const bool pred_ok = consistent && dev < ROOT_STOP_DEV;
            const bool ahead_ok = look_ahead && consistent && dev_next <= 4.0 * (double)ROOT_X_TOL;
            if (resid < stop_resid || pred_ok || ahead_ok) st = ST_LAST;
        }
    }
    if (threadIdx.x == 0) {
        if (!final_pass && (st == ST_RUN || st == ST_LAST)) {
            S.iters += 1;
            S.xloc = (k + 1) & 1;      // X after k + 1 updates: 1 = workspace buffer, 0 = the caller's X
        }
        if (final_pass && (st == ST_RUN || st == ST_LAST)) S.info = ASTERIA_INFO_NOT_CONVERGED;
        if (!final_pass && st == ST_RUN) {
            // iteration k will produce M_{k+1} = f(M_k) and T_{k+1}: advance the spectrum interval
            // through the scalar map and pick the coefficients of T_{k+1} for that new interval
            // every |mu - 1| is at most the measured ||M_k - I||_F: tighten the predicted interval
            double lo_k = (double)S.lo, hi_k = (double)S.hi;
            const double rb = (double)S.resid * 1.001 + 1e-5;
            if (1.0 - rb > lo_k) lo_k = 1.0 - rb;
            if (1.0 + rb < hi_k) hi_k = 1.0 + rb;
            if (!(hi_k > lo_k)) { lo_k = 1.0 - rb; hi_k = 1.0 + rb; }
            const RootInterval im = root_image(lo_k, hi_k, root, (double)S.ca, (double)S.cg);
            double a, g;
            root_coefficients(im.lo, im.hi, root, adapted != 0, ROOT_THETA, a, g);
            S.lo_cur = S.lo; S.hi_cur = S.hi; S.cg_cur = S.cg;
            S.lo = (float)im.lo; S.hi = (float)im.hi;
            S.ca = (float)a; S.cg = (float)g;
            S.coef_next[0] = (float)a; S.coef_next[1] = (float)g;
        }
        state[f] = st;
    }
}

// Copy X from the workspace buffer to the caller's X where the last fp32 update landed there,
// and publish the per-factor outcome.  One workgroup per 128 x 128 tile.
__global__ __launch_bounds__(256) void root_finalize_kernel(const FactorDev *fd, const FactorScal *fs,
                                                            const int *state, int nf, const int *sq_tile_start,
                                                            int first, int32_t *info, int32_t *iters,
                                                            float *resid, float *lambda_max)
{
    int lo = 0, hi = nf - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (sq_tile_start[mid] <= (int)blockIdx.x) lo = mid; else hi = mid - 1;
    }
    const FactorDev &F = fd[lo];
    const FactorScal &S = fs[lo];
    const int lt = (int)blockIdx.x - sq_tile_start[lo];
    if (lt == 0 && threadIdx.x == 0) {
        if (info) info[first + lo] = S.info;
        if (iters) iters[first + lo] = S.iters;
        if (resid) resid[first + lo] = S.resid;
        if (lambda_max) lambda_max[first + lo] = S.lam;
    }
    if (state[lo] == ST_FAIL || S.xloc == 0) return;
    const int n = F.n;
    const int tpr = (n + BN - 1) / BN;
    const int ti = lt / tpr, tj = lt % tpr;
    for (int e = threadIdx.x; e < BM * BN; e += 256) {
        const int row = ti * BM + e / BN, col = tj * BN + e % BN;
        if (row >= n || col >= n) continue;
        F.Xout[(size_t)row * F.ldx + col] = F.X32b[(size_t)row * F.ld32 + col];
    }
}

// ---- host side -------------------------------------------------------------------------------
inline int ld4(int n) { return (n + 3) & ~3; }
inline int ld2(int n) { return (n + 1) & ~1; }

struct Plan {
    int max_iters;
    int fp64_iters;
    int power_iters;
    int root;
    int lowp_from;     // first iteration that may run on the fp16 matrix cores (operands split in two fp16 terms)
    float stop_resid, power_tol, margin;
    bool use64, use32, adapted, lowp_auto;
    int i8_slices;     // 0, or the number of int8 slices the products of the fp64 iterations are computed with
    bool xt_lowp;      // fully automatic precision: X updates on the fp16 cores (split operands) from the
                       // first product on, and the look-ahead stop rule (accuracy class 1e-3)
    LanczosWaits waits;
};

// Host mirror of the device-side schedule for a spectrum of M_0 in [lo0, 1]:
//   *iters  worst-case number of X updates: iterations until sqrt(n) * max|1 - mu| < stop over the
//           interval, plus the last update that follows;
//   *lead64 number of leading iterations that start while the bottom of the spectrum is still
//           below `thr` (those run in fp64 under the automatic precision rule).
// bottom of M's spectrum from which the 16-bit-split tier may run under the automatic rule
constexpr double ROOT_LOWP_FLOOR = 0.5 * 5.96e-8 / 1e-3;

void simulate_schedule(double lo0, int n, int root, bool adapted, double stop, double thr, int cap,
                       int *iters, int *lead64, double thr_lowp = 0.0, int *lead_full = nullptr)
{
    double lo = lo0, hi = 1.0;
    int k = 0, lead = 0, leadf = 0;
    while (k < cap) {
        const double dev = std::max(fabs(1.0 - lo), fabs(1.0 - hi));
        if (sqrt((double)n) * dev < stop) break;
        if (lo < thr) lead = k + 1;
        if (lo < thr_lowp) leadf = k + 1;
        double a, g;
        root_coefficients(lo, hi, root, adapted, ROOT_THETA, a, g);
        const RootInterval im = root_image(lo, hi, root, a, g);
        lo = im.lo; hi = im.hi;
        ++k;
    }
    *iters = k + 1;
    *lead64 = lead;
    if (lead_full) *lead_full = leadf;
}

// The fp32 work matrices of the M-chain (M x 2, T^4) are first written when the fp64 tier hands over - M
// by the epilogue of its last M-update, which no longer stores the fp64 T that lies there - and the
// fp64 T and T^4 are dead from then on: they share one region.
size_t shared_region_bytes(int n, bool use64, bool use32)
{
    const size_t b32 = use32 ? 3 * Carver::need((size_t)n * ld4(n), sizeof(float)) : 0;
    const size_t b64 = use64 ? 2 * Carver::need((size_t)n * ld2(n), sizeof(double)) : 0;
    return b32 > b64 ? b32 : b64;
}

size_t factor_matrix_bytes(int n, bool use64, bool use32)
{
    size_t b = 2 * Carver::need((size_t)n * ld4(n), sizeof(float));            // second X buffer, T (fp32)
    b += shared_region_bytes(n, use64, use32);                                 // fp64 T, T^4 | fp32 M x 2, T^4
    if (use64) b += 2 * Carver::need((size_t)n * ld2(n), sizeof(double));      // fp64 M x 2
    return b;
}

// sliced operands of the int8 path: two buffers of planes, row exponents and diagonals
size_t factor_i8_bytes(int n, int ns)
{
    if (ns <= 0) return 0;
    return 2 * (Carver::need(i8_plane_bytes(n, ns), 1) + Carver::need(i8_rows(n), sizeof(int)) +
                Carver::need(i8_rows(n), sizeof(double))) + Carver::need(1, sizeof(I8Factor));
}

// vectors, partial sums and tables of one factor that both paths need
size_t factor_small_bytes(int n)
{
    const int pmb = (n + LZ_ROWS - 1) / LZ_ROWS;
    return 3 * Carver::need((size_t)ld4(n), sizeof(float)) + Carver::need(2 * (size_t)pmb, sizeof(float)) +
           Carver::need((size_t)pmb, sizeof(double2)) + Carver::need((size_t)tri_tiles(n) * PM_TILE_WORDS, sizeof(float)) +
           sizeof(FactorDev) + sizeof(FactorScal) + 2 * sizeof(int);
}
// ... and those of the fp32 / fp64 path alone
size_t factor_table_bytes(int n) { return Carver::need(2 * (size_t)tri_tiles(n), sizeof(float)) + 16 * sizeof(GemmProblem); }

size_t fixed_bytes() { return 40 * 256; }   // alignment slack of the arrays that hold an entry per factor or tile (24 at most)

asteria_status make_plan(const asteria_root_opts *opts_in, asteria_eps_mode mode, const float *eps,
                         int eps_count, int root, Plan &pl)
{
    asteria_root_opts o;
    asteria_root_opts_default(&o);
    if (opts_in) o = *opts_in;
    if (o.max_iters <= 0 || o.power_iters <= 0) return ASTERIA_INVALID_ARG;
    if (!(o.stop_resid > 0.0f) || !(o.power_tol > 0.0f) || !(o.lambda_margin >= 0.0f)) return ASTERIA_INVALID_ARG;
    if (o.schedule != 0 && o.schedule != 1) return ASTERIA_UNSUPPORTED;
    pl.adapted = o.schedule == 1;
    pl.root = root;
    pl.max_iters = o.max_iters;
    pl.power_iters = o.power_iters;
    pl.stop_resid = o.stop_resid;
    pl.power_tol = o.power_tol;
    pl.margin = o.lambda_margin;
    int j = o.fp64_iters;
    if (j < 0) {
        // fp32 round-off of relative size u injected while the bottom of M's spectrum is mu costs
        // about u / mu in the root: stay in fp64 while 0.5 u_fp32 / mu > 1e-3, i.e. mu < 3e-5.
        if (mode == ASTERIA_EPS_RELATIVE && eps) {
            float emin = eps[0];
            for (int i = 1; i < eps_count; ++i) emin = std::min(emin, eps[i]);
            // the device starts the interval at half of eps s (round-off in the statistics may push
            // eigenvalues slightly below zero): the same start here and in the rule for lowp_from below
            const double lo0 = 0.5 * (double)emin / (1.0 + (double)pl.margin + (double)emin);
            int it = 0;
            if (emin > 0.0f) simulate_schedule(lo0, 1, root, pl.adapted, 1e-3, ROOT_LOWP_FLOOR, o.max_iters, &it, &j);
            else j = o.max_iters;
        } else {
            j = pl.adapted ? 2 : 4;   // the host cannot see eps / lambda_max here
        }
    }
    // Iterations after the fp64 prefix: products of fp32 operands split into two fp16 terms (three
    // fp16 MFMA passes) keep the operands to 2^-22, within a factor 4 of fp32, and run twice as fast
    // as the fp32 matrix cores; they take over as soon as the bottom of M's spectrum is above
    // ROOT_LOWP_FLOOR, the bound below which the automatic rule keeps fp64.
    int jl = o.lowp_from;
    if (jl < 0) {
        jl = o.max_iters;
        if (mode == ASTERIA_EPS_RELATIVE && eps) {
            float emin = eps[0];
            for (int i = 1; i < eps_count; ++i) emin = std::min(emin, eps[i]);
            if (emin > 0.0f) {
                const double lo0 = 0.5 * (double)emin / (1.0 + (double)pl.margin + (double)emin);
                int it = 0, l64 = 0;
                simulate_schedule(lo0, 1, root, pl.adapted, 1e-3, 0.0, o.max_iters, &it, &l64, ROOT_LOWP_FLOOR, &jl);
            }
        }
    }
    pl.lowp_from = jl;
    pl.lowp_auto = o.lowp_from < 0;
    // only under fully automatic precision rules, and only where they use the 16-bit tier at all
    pl.xt_lowp = pl.lowp_auto && o.fp64_iters < 0 && jl < o.max_iters;
    pl.fp64_iters = std::min(j, pl.max_iters);
    pl.use64 = pl.fp64_iters > 0;
    pl.use32 = pl.fp64_iters < pl.max_iters;
    if (o.int8_slices != -1 && o.int8_slices != 0 && o.int8_slices != 4 && o.int8_slices != 5) return ASTERIA_UNSUPPORTED;
    pl.i8_slices = pl.use64 ? (o.int8_slices < 0 ? 5 : o.int8_slices) : 0;
    return ASTERIA_OK;
}

asteria_status validate(const asteria_factor *f, int nf, int root, const float *eps, int eps_count)
{
    if (!f || nf <= 0 || !eps) return ASTERIA_INVALID_ARG;
    if (root != 2 && root != 4) return ASTERIA_UNSUPPORTED;
    if (eps_count != 1 && eps_count != nf) return ASTERIA_INVALID_ARG;
    for (int i = 0; i < eps_count; ++i)
        if (!(eps[i] >= 0.0f) || !(eps[i] < 3.0e38f)) return ASTERIA_INVALID_ARG;
    for (int i = 0; i < nf; ++i) {
        if (!f[i].A || !f[i].X || f[i].n <= 0 || f[i].ldx < f[i].n) return ASTERIA_INVALID_ARG;
        if (f[i].a_layout == ASTERIA_LAYOUT_FULL) { if (f[i].lda < f[i].n) return ASTERIA_INVALID_ARG; }
        else if (f[i].a_layout == ASTERIA_LAYOUT_PACKED) { if (reinterpret_cast<uintptr_t>(f[i].A) & 15u) return ASTERIA_INVALID_ARG; }
        else return ASTERIA_INVALID_ARG;
    }
    return ASTERIA_OK;
}

// The grouped-GEMM problem tables of one pass: [parity] X' = X T on the fp32 buffers, and
// [precision 0 = fp32, 1 = fp64][parity][T T | T^2 T^2 | T^p M] for the chain of M.
struct RootTables {
    GemmProblem *xt[2];
    GemmProblem *tab[2][2][3];
    GemmProblem *last64[2];    // [parity] the M-update of the last fp64 iteration: it hands M over in fp32
};

// one thread per factor writes its entry of every table
__global__ void root_tables_kernel(const FactorDev *__restrict__ fd, FactorScal *fs, int cnt, int root, int use32,
                                   int use64, RootTables rt, const I8Factor *xf)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= cnt) return;
    const FactorDev F = fd[i];
    const float ca = (float)(root + 1) / (float)root, cg = 1.0f / (float)root;
    GemmProblem p = {};
    p.M = p.N = p.K = F.n;
    p.state_idx = i;
    p.alpha = 1.0f; p.beta = 0.0f; p.ep_a = ca; p.ep_g = cg;
    p.flags = GEMM_SYM;
    p.tile_start = F.tile_start;
    p.sa = ROOT_F16_SCALE; p.sb = ROOT_F16_SCALE;       // read by the fp16-split kernel only
    for (int pa = 0; pa < 2; ++pa) {
        // X after an odd number of updates lives in the workspace buffer, else in the caller's X
        GemmProblem q = p;
        q.state_mask = (1 << ST_RUN) | (1 << ST_LAST);
        q.A = pa ? (const void *)F.X32b : (const void *)F.Xout; q.lda = pa ? F.ld32 : F.ldx;
        q.B = F.T32; q.ldb = F.ld32;
        q.C = pa ? (void *)F.Xout : (void *)F.X32b; q.ldc = pa ? F.ldx : F.ld32;
        q.sa_dev = &fs[i].x_scale;
        rt.xt[pa][i] = q;
    }
    p.state_mask = (1 << ST_RUN);
    for (int pr = 0; pr < 2; ++pr) {
        if ((pr == 0 && !use32) || (pr == 1 && !use64)) continue;
        for (int pa = 0; pa < 2; ++pa) {
            const void *Tm, *Mcur;
            void *Mnext, *T4, *Tw;
            int ldw;
            if (pr == 1) {
                Tm = F.T64; Tw = F.T64; Mcur = F.M64[pa]; Mnext = F.M64[pa ^ 1]; T4 = F.T464; ldw = F.ld64;
            } else {
                Tm = F.T32; Tw = F.T32; Mcur = F.M32[pa]; Mnext = F.M32[pa ^ 1]; T4 = F.T432; ldw = F.ld32;
            }
            GemmProblem q = p;
            // with the int8 path on, the fp64 launches take the products it declines
            if (pr == 1 && xf) q.gate = &xf[i].gate;
            // launch 0: T2 = T T, kept in the buffer that receives M' afterwards (root 4) or in
            // the T^4 buffer (root 2, where the M-update reads T2 while writing M')
            void *T2 = (root == 4) ? Mnext : T4;
            q.A = Tm; q.lda = ldw; q.B = Tm; q.ldb = ldw; q.C = T2; q.ldc = ldw;
            rt.tab[pr][pa][0][i] = q;
            // launch 1: T4 = T2 T2 (root 4 only)
            q.A = T2; q.B = T2; q.C = T4;
            rt.tab[pr][pa][1][i] = q;
            // launch 2: M' = T^p M, T' = a I - g M' (+ its fp32 copy in the fp64 tier), residual partial sums
            q.A = (root == 4) ? (const void *)T4 : (const void *)T2; q.B = Mcur;
            q.C = Mnext; q.C2 = Tw; q.ldc2 = ldw; q.partial = F.partial;
            if (pr == 1) { q.C3 = F.T32; q.ldc3 = F.ld32; }
            q.coef = fs[i].coef_next;
            q.flags = GEMM_SYM | GEMM_EPI_ROOT;
            rt.tab[pr][pa][2][i] = q;
            if (pr == 1 && use32) {
                // ... and when it is the last fp64 iteration: the fp64 M' and T' would never be read, the fp32
                // tier starts from M' in the buffer its parity expects (it lies over the fp64 T, which this
                // product does not read)
                q.flags |= GEMM_EPI_HANDOVER;
                q.C4 = F.M32[pa ^ 1]; q.ldc4 = F.ld32;
                rt.last64[pa][i] = q;
            }
        }
    }
}

// Compute units that work on a stream can use, 0 where that cannot be found out.
int stream_cus(hipStream_t stream)
{
    uint32_t mask[32] = {};
    if (hipExtStreamGetCUMask(stream, 32, mask) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    int cus = 0;
    for (uint32_t w : mask) cus += __builtin_popcount(w);
    return cus;
}

// Whether the lambda_max estimate of a pass keeps its matrices in registers of several workgroups: wherever they fit and find room side by
// side, except for factors that one workgroup holds by itself.  The whole refresh in us, by the ways below / so, taken in turn: 3 blocks of 777 x 1000 in
// blocks of 512, evenly dense spectra 1621 / 1265; 6 of 1000 x 333 1106 / 1036; 1 of 512 x 400 487 / 406; 1 of 1024 x 1024 712 / 654; 100 of
// 512 x 300 3811 / 3802; 64 of 1024 x 1024 16837 / 15807; 3 of 2000 x 1500 4001 / 3876; the 1.1B model 248.7 / 243.2 ms, packed 251.6 / 243.7.
bool lanczos_by_cluster(int n_max, hipStream_t stream) { return n_max > 256 && n_max <= LC_MAX_N && lanczos_cluster_room(n_max, stream_cus(stream)); }

// The others (larger factors, little room, the general path).  Small factors, and batches that keep every CU busy until the
// largest factor is done: one workgroup per factor, one launch.  Otherwise one launch per step - 32 of them, then one
// workgroup per factor takes what has not settled; from n = 2048 on launches throughout.
// General path with one fp32 iteration, us, launches of steps / a workgroup per factor, power-law spectrum (8 steps):
//   1 factor    n = 320 309 / 298, 448 328 / 347, 512 322 / 340, 640 368 / 452, 768 390 / 507 (packed ones need three launches a step)
//   n = 1024    64 factors 2790 / 2871, 128 5295 / 5147, 192 7830 / 7475, 256 10367 / 9777
//   200 factors of n = 128 and one of 4096: 4326 / 10584 (evenly spaced spectrum, 128 steps: 7701 / 72139), which is
//   why the rule counts elements against those of the largest factor
// 32 launches and a workgroup / launches throughout: power law n = 320 309 / 491, 1024 446 / 636, 1536 572 / 763, 2000 844 / 1021, 3000 1832 /
// 1849; evenly spaced n = 512 1224 / 1020, 1024 1955 / 1147, 1536 5916 / 1568, 2000 14702 / 2314: most spectra settle within the 32.
bool lanczos_by_factor(double elems, int n_max, bool any_packed)
{
    return n_max <= LZ_WG_N || (elems >= (double)LZ_WG_BATCH * n_max * n_max && n_max <= LZ_WG_MAX_N && !any_packed);
}
constexpr int LZ_LAUNCHES = 32, LZ_LAUNCH_N = 2048;

asteria_status lambda_max_launches(const FactorDev *d_fd, FactorScal *d_fs, int cnt, double elems, const Plan &pl, bool any_full, bool any_packed,
                                   int tri_max, int n_max, hipStream_t stream, int cluster_total = 0, uint2 *cluster_map = nullptr,
                                   int *cluster_ticket = nullptr)      // workgroups of lanczos_cluster_kernel (two words), 0: one of the other ways
{
    const int steps = std::min(pl.power_iters, LZ_MAX);
    const float tol2 = pl.power_tol * pl.power_tol;
    const int ld = (n_max + 255) & ~255;
    const size_t lds = 3 * (size_t)ld * sizeof(float);
    static bool cfg_f[MAX_DEVICES] = {}, cfg_s[MAX_DEVICES] = {};
    if (cluster_total > 0) {
        hipLaunchKernelGGL(lanczos_prepare_kernel, dim3(cnt), dim3(256), 0, stream, d_fd, d_fs, cluster_map, cluster_ticket);
        hipLaunchKernelGGL(lanczos_cluster_kernel, dim3(cluster_total), dim3(LC_THREADS), 0, stream, d_fd, d_fs, cluster_map, cluster_ticket, tol2, steps,
                           pl.waits);
        ASTERIA_HIP_TRY(hipGetLastError());
        return ASTERIA_OK;
    }
    if (lanczos_by_factor(elems, n_max, any_packed)) {
        if (any_packed) hipLaunchKernelGGL(lanczos_unpack_kernel, dim3(tri_max, cnt), dim3(256), 0, stream, d_fd);
        if (n_max <= LZ_FEW_N) {
            hipLaunchKernelGGL((lanczos_factor_kernel<true, LZ_FEW_THREADS>), dim3(cnt), dim3(LZ_FEW_THREADS), lds, stream, d_fd, d_fs, tol2, steps, -1, ld);
        } else if (n_max <= 256) {
            hipLaunchKernelGGL(lanczos_factor_kernel<true>, dim3(cnt), dim3(LZ_THREADS), lds, stream, d_fd, d_fs, tol2, steps, -1, ld);
        } else {
            ASTERIA_HIP_TRY(ensure_dynamic_lds(reinterpret_cast<const void *>(lanczos_factor_kernel<false>), 3 * sizeof(float) * LZ_WG_MAX_N, cfg_f));
            hipLaunchKernelGGL(lanczos_factor_kernel<false>, dim3(cnt), dim3(LZ_THREADS), lds, stream, d_fd, d_fs, tol2, steps, -1, ld);
        }
        ASTERIA_HIP_TRY(hipGetLastError());
        return ASTERIA_OK;
    }
    if (!any_packed && n_max <= 16384) {
        const int blocks = (n_max + LZ_ROWS - 1) / LZ_ROWS;
        const size_t lds1 = (size_t)ld * sizeof(float);
        ASTERIA_HIP_TRY(ensure_dynamic_lds(reinterpret_cast<const void *>(lanczos_step_kernel), 16384 * sizeof(float), cfg_s));
        const int launches = n_max < LZ_LAUNCH_N ? std::min(steps, LZ_LAUNCHES) : steps;
        for (int j = 0; j < launches; ++j)
            hipLaunchKernelGGL(lanczos_step_kernel, dim3(blocks + 1, cnt), dim3(256), lds1, stream, d_fd, d_fs, tol2, j, blocks);
        // the last launch's y is in place, its alpha is not: one workgroup per factor goes on from there, or
        // (no steps left) a launch of the workgroup that keeps the recurrence alone
        if (launches == steps) {
            hipLaunchKernelGGL(lanczos_step_kernel, dim3(1, cnt), dim3(256), lds1, stream, d_fd, d_fs, tol2, steps, 0);
        } else {
            ASTERIA_HIP_TRY(ensure_dynamic_lds(reinterpret_cast<const void *>(lanczos_factor_kernel<false>), 3 * sizeof(float) * LZ_WG_MAX_N, cfg_f));
            hipLaunchKernelGGL(lanczos_factor_kernel<false>, dim3(cnt), dim3(LZ_THREADS), lds, stream, d_fd, d_fs, tol2, steps, launches, ld);
        }
        ASTERIA_HIP_TRY(hipGetLastError());
        return ASTERIA_OK;
    }
    hipLaunchKernelGGL(pm_init_kernel, dim3(cnt), dim3(256), 0, stream, d_fd, d_fs);
    for (int it = 0; it < steps; ++it) {
        // the three vectors rotate: v_j in src, A v_j (then v_{j+1}) in dst, v_{j-1} in prev
        const int src = it % 3, dst = (it + 1) % 3, prev = (it + 2) % 3, first = it == 0 ? 1 : 0;
        if (any_full)
            hipLaunchKernelGGL(pm_matvec_kernel, dim3((n_max + LZ_ROWS - 1) / LZ_ROWS, cnt), dim3(256), 0, stream, d_fd, d_fs, src, dst, first);
        if (any_packed) {
            hipLaunchKernelGGL(pm_packed_tile_kernel, dim3(tri_max, cnt), dim3(256), 0, stream, d_fd, d_fs, src, first);
            hipLaunchKernelGGL(pm_packed_reduce_kernel, dim3((n_max + PACK_T - 1) / PACK_T, cnt), dim3(PACK_T), 0, stream, d_fd, d_fs, src, dst, first);
        }
        hipLaunchKernelGGL(pm_lanczos_kernel, dim3(cnt), dim3(256), 0, stream, d_fd, d_fs, tol2, it, src, dst, prev, first, it + 1 == steps ? 1 : 0);
    }
    ASTERIA_HIP_TRY(hipGetLastError());
    return ASTERIA_OK;
}

}  // namespace
#include "root_plane_path.h"
namespace {

// The plane path serves the fully automatic precision rules; everything pinned, absolute eps, square roots and
// the classical schedule take run_pass below.
bool plane_path(const Plan &pl, asteria_eps_mode mode, int n_max)
{
    return pl.xt_lowp && mode == ASTERIA_EPS_RELATIVE && pl.root == 4 && pl.adapted && n_max <= 16384;
}

// Whether a factor's digits can turn out too coarse (largest possible diagonal of M_0: 1)
bool plane_needs_f64(const Plan &pl, double lo0, int n_max)
{
    if (pl.fp64_iters <= 0) return false;
    if (pl.i8_slices < 5 || digit_rounding(n_max, 5, 1.0, lo0) > DIGIT_ROUNDING) return true;
    // E2 <= a^2 <= 2^4 on M and W <= 2^1 with 6 levels of 5 digits, against a bottom lifted at least tenfold
    return (1.0 + 16.0) * digit_dropped(n_max, 5, 6, 4, 1) / (10.0 * lo0) > DIGIT_DROPPED;
}

asteria_status run_pass_planes(const asteria_factor *f, int first, int cnt, const float *eps, int eps_count, const Plan &pl, bool f64,
                               int32_t *info, int32_t *iters, float *resid, float *lambda_max, void *ws, hipStream_t stream)
{
    Carver cv(ws);
    FactorDev *d_fd = cv.take<FactorDev>(cnt);
    FactorScal *d_fs = cv.take<FactorScal>(cnt);
    int *d_state = cv.take<int>(cnt);
    int *d_flags = cv.take<int>(cnt);
    std::vector<FactorDev> fd(cnt);
    int tri_total = 0, tri64_total = 0, tri256_total = 0, tri_max = 0, n_max = 0;
    double work128 = 0.0, work256 = 0.0, rows = 0.0;
    bool any_packed = false, any_full = false;
    double a_min = 1.0, elems = 0.0;
    const bool prefix = pl.fp64_iters > 0;
    int cluster_total = 0;
    for (int i = 0; i < cnt; ++i) {
        const asteria_factor &a = f[first + i];
        FactorDev &F = fd[i];
        memset(&F, 0, sizeof(F));
        const int n = a.n;
        n_max = std::max(n_max, n);
        elems += (double)n * n;
        F.A = a.A; F.Xout = a.X; F.n = n; F.lda = a.lda; F.ldx = a.ldx;
        F.rowb = pair_row_bytes(n); F.ld64 = ld2(n);
        F.ntri = tri_tiles(n);
        F.tile_start = tri_total; tri_total += F.ntri;
        tri64_total += tri_tiles_of(n, 64); tri256_total += tri_tiles_of(n, 256);
        work128 += pair_work(n, 128); work256 += pair_work(n, 256); rows += n;
        F.npart = plane_partials(n);
        F.flags = d_flags + i;
        F.a_packed = a.a_layout == ASTERIA_LAYOUT_PACKED ? 1 : 0;
        F.pm_blocks = F.a_packed ? (n + PACK_T - 1) / PACK_T : (n + LZ_ROWS - 1) / LZ_ROWS;
        F.Aw = a.A; F.ldw = a.lda;
        if (F.a_packed) { any_packed = true; tri_max = std::max(tri_max, F.ntri); }
        else any_full = true;
        F.lz_start = cluster_total; cluster_total += lanczos_members(n);
        F.eps_in = eps[eps_count == 1 ? 0 : first + i];
        const double er = (double)F.eps_in;
        a_min = std::min(a_min, er / (1.0 + (double)pl.margin + er));
        for (int v = 0; v < 3; ++v) F.pv[v] = cv.take<float>(ld4(n));
        F.pm_partial = cv.take<float>(2 * (size_t)((n + LZ_ROWS - 1) / LZ_ROWS));
        F.pm_partial2 = cv.take<double2>((n + LZ_ROWS - 1) / LZ_ROWS);
        F.pm_tile = cv.take<float>((size_t)F.ntri * PM_TILE_WORDS);
        F.partial = cv.take<float>(F.npart);
        F.qpart = cv.take<float>(F.npart);
        const size_t pair = plane_pair_bytes(n), slot = prefix ? plane_slot_bytes(n, f64) : pair;
        for (int v = 0; v < 2; ++v) F.X[v] = cv.take<char>(pair);
        // X_0 is never written: a full copy of packed statistics and two vectors of the estimate lie there
        if (F.a_packed) { F.Aw = reinterpret_cast<const float *>(F.X[0]); F.ldw = F.rowb / 4; }
        for (int v = 0; v < 2; ++v) F.py[v] = reinterpret_cast<float *>(F.X[0]) + v * ld4(n);
        F.lz_words = reinterpret_cast<uint64_t *>(F.X[0]);     // (16 n + 32 bytes a member; a row of X_0 alone has 128)
        char *chain[4] = {nullptr, nullptr, cv.take<char>(std::max(slot, 2 * pair)), cv.take<char>(slot)};
        if (prefix)
            for (int v = 0; v < 4; ++v) {
                if (v < 2) chain[v] = cv.take<char>(slot);
                F.D[v] = chain[v]; F.F[v] = reinterpret_cast<double *>(chain[v]);
            }
        F.P[0] = chain[2]; F.P[1] = chain[2] + pair; F.P[2] = F.P[3] = chain[3];
    }
    const int edge = pair_tile_edge(tri64_total, tri_total, tri256_total, tri_tiles(n_max), work128, work256, rows / cnt);
    int pair_total = 0;
    for (FactorDev &F : fd) { F.tile_start_p = pair_total; pair_total += tri_tiles_of(F.n, edge); }
    // (until the tiles are written there d_map holds the members of lanczos_cluster_kernel, fewer than tiles, and d_state, with room for 64, its two words)
    uint2 *d_map = cv.take<uint2>(tri_total), *d_map_p = edge == 128 ? d_map : cv.take<uint2>(pair_total);
    PlaneF64Tables ft = {};
    if (f64)
        for (int o = 0; o < 4; ++o) ft.t[o] = cv.take<GemmProblem>(cnt);

    // degrees of T by iteration and the iteration budget: the sequence for the smallest eps, then a few more for a
    // factor whose spectrum left the interval the sequence is made for
    const double lo0 = 0.5 * a_min;
    std::vector<int> deg;
    if (pl.fp64_iters <= 2) {
        for (const char *q = root_degrees(lo0 / ROOT_TOP); *q; ++q) deg.push_back(*q - '0');
    } else {
        // a longer prefix is linear, and so is the rest but for the last two: degrees 2 and 3 take one product less
        // than three linear ones and leave a tenth of their truncation (eps = 1e-8: 3.4e-4 of X after 10 linear, 2e-5)
        RootInterval I = {lo0, ROOT_TOP};
        for (int k = 0; k + 2 < pl.max_iters && deg.empty(); ++k) {
            if (k >= pl.fp64_iters) {
                const RootInterval two = root_poly(I.lo, I.hi, 2).image, three = root_poly(two.lo, two.hi, 3).image;
                if (std::max(1.0 - three.lo, three.hi - 1.0) <= 4.0 * (double)ROOT_X_TOL) {
                    deg.assign(k, 1);
                    deg.push_back(2); deg.push_back(3);
                }
            }
            I = root_poly(I.lo, I.hi, 1).image;
        }
    }
    int K;
    if (!deg.empty()) {
        for (int e = 0; e < 3; ++e) deg.push_back(2);
        K = (int)deg.size();
    } else {
        int it = 0, lead = 0;
        simulate_schedule(lo0, n_max, 4, true, (double)pl.stop_resid, 0.0, pl.max_iters, &it, &lead);
        K = it + 2;
    }
    K = std::min(K, pl.max_iters);
    deg.resize(K + 1, 1);
    const int J = std::min(pl.fp64_iters, K);
    const bool linear0 = deg[0] == 1;

    ASTERIA_HIP_TRY(upload_async(d_fd, fd.data(), sizeof(FactorDev) * cnt, stream));
    if (f64)
        hipLaunchKernelGGL(plane_f64_tables_kernel, dim3((cnt + 127) / 128), dim3(128), 0, stream, d_fd, d_fs, cnt, linear0 ? 1 : 0, ft);
    const bool by_cluster = lanczos_by_cluster(n_max, stream);
    ASTERIA_TRY(lambda_max_launches(d_fd, d_fs, cnt, elems, pl, any_full, any_packed, tri_max, n_max, stream, by_cluster ? cluster_total : 0, d_map,
                                    d_state));

    // intervals and T of a factor that follows the schedule (the device works in fp32 for the scaling: 1e-5 of slack)
    std::vector<PlaneControl> ctl(K + 1);
    {
        double lo = lo0 * (1.0 - 1e-5), hi = ROOT_TOP;
        for (int k = 0; k <= K; ++k) {
            ctl[k].lo = lo; ctl[k].hi = hi;
            ctl[k].T = root_poly(lo, hi, deg[k]);
            lo = ctl[k].T.image.lo; hi = ctl[k].T.image.hi;
        }
    }
    auto control = [&](int k) {
        PlaneControl &c = ctl[k];
        c.k = k; c.degree = deg[k]; c.next_linear = (k + 1 < K && deg[k + 1] == 1) ? 1 : 0;
        c.prefix = J; c.wide_next = (k + 1 < J && deg[k + 1] <= 2) ? 1 : 0;
        c.digits_max = pl.i8_slices; c.final_pass = k == K ? 1 : 0; c.stop_resid = pl.stop_resid;
        c.counters = profile_i8_counters();
        return c;
    };
    hipLaunchKernelGGL(plane_setup_kernel, dim3(cnt), dim3(256), 0, stream, d_fd, d_fs, d_state, pl.margin, control(0), d_map,
                       edge == 128 ? nullptr : d_map_p, edge, pl.power_tol * pl.power_tol, by_cluster ? std::min(pl.power_iters, LZ_MAX) : 0);
    hipLaunchKernelGGL(plane_init_kernel, dim3(tri_total, 4), dim3(256), 0, stream, d_fd, d_fs, d_state, d_map, linear0 ? 1 : 0);
    ASTERIA_HIP_TRY(hipGetLastError());
    for (int k = 0; k < K; ++k) {
        if (k > 0) hipLaunchKernelGGL(plane_control_kernel, dim3(cnt), dim3(64), 0, stream, d_fd, d_fs, d_state, control(k));
        const int d = deg[k];
        const bool pre = k < J;
        auto pair = [&](int op0, int op1) -> hipError_t {
            switch (edge) {
            case 64: return launch_pair_product<2, 2, 2, 2, 4>(d_fd, d_fs, d_state, d_map_p, pair_total, op0, op1, k, d, stream);
            case 128:
                // one workgroup per CU at most: eight wavefronts hide more of each other's waits than four; with two workgroups per CU four
                // are better.  Refresh in us, eight / four, by tiles: n = 1024 216 1007 / 1079, 288 1572 / 1454, 360 1684 / 1557, 504 1991 /
                // 1812; n = 333 240 726 / 757, 300 1052 / 984; n = 512 400 1321 / 1199; n = 2048 and 64 274 2526 / 2355
                if ((op1 >= 0 ? 2 : 1) * pair_total <= PLANE_CUS)
                    return launch_pair_product<4, 2, 2, 4, 4>(d_fd, d_fs, d_state, d_map_p, pair_total, op0, op1, k, d, stream);
                return launch_pair_product<2, 2, 4, 4, 2>(d_fd, d_fs, d_state, d_map_p, pair_total, op0, op1, k, d, stream);
            default: return launch_pair_product<4, 2, 4, 8, 2>(d_fd, d_fs, d_state, d_map_p, pair_total, op0, op1, k, d, stream);
            }
        };
        auto from_f64 = [&](int what) {
            if (f64)
                hipLaunchKernelGGL(plane_from_f64_kernel, dim3((unsigned)(((size_t)n_max * plane_groups(n_max) * 2 + 255) / 256), (unsigned)cnt),
                                   dim3(256), 0, stream, d_fd, d_fs, d_state, k, what);
        };
        // a product of the chain in every storage it can be in, and a second one on pair planes; planes: what is made of the fp64 result
        auto product = [&](int op, int tab, int op1, int planes) -> hipError_t {
            hipError_t e = hipSuccess;
            if (pre && f64) {
                e = launch_gemm_grouped<double, double, double, false, false>(ft.t[tab], cnt, tri_total, d_state, stream);
                if (planes >= 0) from_f64(planes);
            }
            // One launch for either number of digits, refresh in us, one / one each (both in quarters up to PLANE_QUARTERS), by halves of tiles:
            // n = 128 720 873 / 890, n = 1024 432 1006 / 1019, 720 1531 / 1545, 1152 2297 / 2317, 1728 3159 / 3181, eps = 1e-8 1152 5049 /
            // 5072; n = 512 640 1073 / 1091, 2400 3244 / 3361.  Beside 256-wide tiles within what runs differ by: n = 1024 5760 9758 / 9809,
            // 14400 22961 / 22981, n = 768 at eps = 1e-8 5880 18915 / 18968; there the launches stay apart, as a profile reports them.
            if (e == hipSuccess && pre && pl.i8_slices > 4 && edge != 256) {
                e = 2 * tri_total <= PLANE_QUARTERS
                        ? launch_digit_product<0, true>(d_fd, d_fs, d_state, d_map, tri_total, op, k, d, stream)
                        : launch_digit_product<0>(d_fd, d_fs, d_state, d_map, tri_total, op, k, d, stream);
            } else {
                if (e == hipSuccess && pre && pl.i8_slices > 0) e = launch_digit_product<4>(d_fd, d_fs, d_state, d_map, tri_total, op, k, d, stream);
                if (e == hipSuccess && pre && pl.i8_slices > 4) e = launch_digit_product<5>(d_fd, d_fs, d_state, d_map, tri_total, op, k, d, stream);
            }
            return e == hipSuccess ? pair(op, op1) : e;
        };
        if (pre && k > 0 && pl.i8_slices > 0) from_f64(2);
        if (d == 2) ASTERIA_HIP_TRY(product(OP_SQ, 0, -1, 0));
        if (d == 3) { ASTERIA_HIP_TRY(pair(OP_SQ3, -1)); ASTERIA_HIP_TRY(pair(OP_CUBE, -1)); }
        ASTERIA_HIP_TRY(product(OP_E2, 1, k > 0 ? (int)OP_X : -1, -1));
        ASTERIA_HIP_TRY(product(OP_W, 2, -1, -1));
        ASTERIA_HIP_TRY(product(OP_M, 3, -1, 1));
        ASTERIA_HIP_TRY(hipGetLastError());
    }
    hipLaunchKernelGGL(plane_control_kernel, dim3(cnt), dim3(64), 0, stream, d_fd, d_fs, d_state, control(K));
    hipLaunchKernelGGL(plane_finalize_kernel, dim3(64, (unsigned)cnt), dim3(256), 0, stream, d_fd, d_fs, d_state, first, info, iters, resid, lambda_max);
    ASTERIA_HIP_TRY(hipGetLastError());
    return ASTERIA_OK;
}

// one pass over factors [first, first + cnt)
asteria_status run_pass(const asteria_factor *f, int first, int cnt, int root, asteria_eps_mode mode, const float *eps, int eps_count,
                        const Plan &pl, int32_t *info, int32_t *iters, float *resid, float *lambda_max, void *ws, hipStream_t stream)
{
    Carver cv(ws);
    FactorDev *d_fd = cv.take<FactorDev>(cnt);
    FactorScal *d_fs = cv.take<FactorScal>(cnt);
    int *d_state = cv.take<int>(cnt);
    int *d_sq = cv.take<int>(cnt);
    GemmProblem *d_tab[2][2][3];   // [precision 0 = fp32, 1 = fp64][parity][launch T T | T^2 T^2 | T^p M]
    GemmProblem *d_xt[2];          // [parity] X' = X T on the fp32 buffers (every precision tier)
    for (int pa = 0; pa < 2; ++pa) d_xt[pa] = cv.take<GemmProblem>(cnt);
    for (int pr = 0; pr < 2; ++pr)
        for (int pa = 0; pa < 2; ++pa)
            for (int l = 0; l < 3; ++l) d_tab[pr][pa][l] = cv.take<GemmProblem>(cnt);
    GemmProblem *d_last64[2];      // [parity] M-update of the last fp64 iteration
    for (int pa = 0; pa < 2; ++pa) d_last64[pa] = cv.take<GemmProblem>(cnt);

    std::vector<FactorDev> fd(cnt);
    std::vector<int> sq(cnt);
    int tri_total = 0, sq_total = 0, tri_max = 0;
    bool any_packed = false, any_full = false;
    int n_max = 0;
    double a_min = 1.0, elems = 0.0;
    for (int i = 0; i < cnt; ++i) {
        const asteria_factor &a = f[first + i];
        FactorDev &F = fd[i];
        memset(&F, 0, sizeof(F));
        const int n = a.n;
        n_max = std::max(n_max, n);
        elems += (double)n * n;
        F.A = a.A; F.Xout = a.X; F.n = n; F.lda = a.lda; F.ldx = a.ldx;
        F.ld32 = ld4(n); F.ld64 = ld2(n);
        F.ntri = tri_tiles(n);
        F.tile_start = tri_total; tri_total += F.ntri;
        const int tpr = (n + BM - 1) / BM;
        sq[i] = sq_total; sq_total += tpr * tpr;
        F.a_packed = a.a_layout == ASTERIA_LAYOUT_PACKED ? 1 : 0;
        // partial sums of the mat-vec: per block of LZ_ROWS rows, or per block of 128 rows for packed tiles
        F.pm_blocks = F.a_packed ? (n + PACK_T - 1) / PACK_T : (n + LZ_ROWS - 1) / LZ_ROWS;
        F.Aw = a.A; F.ldw = a.lda;
        if (F.a_packed) { any_packed = true; tri_max = std::max(tri_max, F.ntri); }
        else any_full = true;
        F.eps_in = eps[eps_count == 1 ? 0 : first + i];
        if (mode == ASTERIA_EPS_RELATIVE) {
            const double er = (double)F.eps_in;
            a_min = std::min(a_min, er / (1.0 + (double)pl.margin + er));
        }
        for (int v = 0; v < 3; ++v) F.pv[v] = cv.take<float>(ld4(n));
        F.pm_partial = cv.take<float>(2 * (size_t)((n + LZ_ROWS - 1) / LZ_ROWS));
        F.pm_partial2 = cv.take<double2>((n + LZ_ROWS - 1) / LZ_ROWS);
        F.pm_tile = cv.take<float>((size_t)F.ntri * PM_TILE_WORDS);
        F.partial = cv.take<float>(2 * (size_t)F.ntri);
    }
    // factors too large for exact int32 sums (never reached by the 16384 limit of the other tiers'
    // workloads) keep the fp64 cores
    const int ns8 = (pl.i8_slices > 0 && n_max <= 65536) ? pl.i8_slices : 0;
    I8Factor *d_xf = nullptr;
    std::vector<I8Factor> xfh;
    if (ns8 > 0) {
        d_xf = cv.take<I8Factor>(cnt);
        xfh.resize(cnt);
        for (int i = 0; i < cnt; ++i) {
            I8Factor &X = xfh[i];
            memset(&X, 0, sizeof(X));
            const int n = fd[i].n;
            for (int b = 0; b < 2; ++b) {
                X.planes[b] = cv.take<int8_t>(i8_plane_bytes(n, ns8));
                X.expo[b] = cv.take<int>(i8_rows(n));
                X.diag[b] = cv.take<double>(i8_rows(n));
            }
            X.n = n; X.kb = (n + 31) / 32;
        }
    }
    for (int i = 0; i < cnt; ++i) {
        FactorDev &F = fd[i];
        const size_t e32 = (size_t)F.n * F.ld32, e64 = (size_t)F.n * F.ld64;
        F.X32b = cv.take<float>(e32);
        if (F.a_packed) { F.Aw = F.X32b; F.ldw = F.ld32; }      // room for a full copy while X is not there yet
        F.T32 = cv.take<float>(e32);
        for (int v = 0; v < 2; ++v) F.py[v] = F.T32 + v * ld4(F.n);   // T_0 is not there yet either
        unsigned char *shared = cv.take<unsigned char>(shared_region_bytes(F.n, pl.use64, pl.use32));
        if (pl.use32) {
            const size_t step = Carver::need(e32, sizeof(float));
            F.M32[0] = reinterpret_cast<float *>(shared);
            F.M32[1] = reinterpret_cast<float *>(shared + step);
            F.T432 = reinterpret_cast<float *>(shared + 2 * step);
        }
        if (pl.use64) {
            F.T64 = reinterpret_cast<double *>(shared);
            F.T464 = reinterpret_cast<double *>(shared + Carver::need(e64, sizeof(double)));
            F.M64[0] = cv.take<double>(e64); F.M64[1] = cv.take<double>(e64);
        }
    }

    // iteration budget known on the host
    int K = pl.max_iters;
    if (mode == ASTERIA_EPS_RELATIVE && a_min > 0.0) {
        int it = 0, lead = 0;
        simulate_schedule(a_min * 0.5, n_max, root, pl.adapted, (double)pl.stop_resid, 0.0, pl.max_iters, &it, &lead);
        K = std::min(K, it + 2);
    }
    const int j64 = std::min(pl.fp64_iters, K);
    // checked up to n = 4096; beyond 16384 the automatic rule keeps the factors on the fp32 cores
    const int jlow = (pl.lowp_auto && n_max > 16384) ? K : pl.lowp_from;

    // problem tables: written on the device from the factor descriptors (the 14 tables are 11 times
    // the size of the descriptors, and host tables would travel as kernel arguments)
    ASTERIA_HIP_TRY(upload_async(d_fd, fd.data(), sizeof(FactorDev) * cnt, stream));
    ASTERIA_HIP_TRY(upload_async(d_sq, sq.data(), sizeof(int) * cnt, stream));
    RootTables rt;
    for (int pa = 0; pa < 2; ++pa) rt.xt[pa] = d_xt[pa];
    for (int pr = 0; pr < 2; ++pr)
        for (int pa = 0; pa < 2; ++pa)
            for (int l = 0; l < 3; ++l) rt.tab[pr][pa][l] = d_tab[pr][pa][l];
    for (int pa = 0; pa < 2; ++pa) rt.last64[pa] = d_last64[pa];
    if (ns8 > 0) ASTERIA_HIP_TRY(upload_async(d_xf, xfh.data(), sizeof(I8Factor) * cnt, stream));
    hipLaunchKernelGGL(root_tables_kernel, dim3((cnt + 127) / 128), dim3(128), 0, stream, d_fd, d_fs, cnt, root,
                       pl.use32 ? 1 : 0, pl.use64 ? 1 : 0, rt, d_xf);
    ASTERIA_HIP_TRY(hipGetLastError());

    // 1. lambda_max
    ASTERIA_TRY(lambda_max_launches(d_fd, d_fs, cnt, elems, pl, any_full, any_packed, tri_max, n_max, stream));
    const int ctl_blocks = (cnt + 127) / 128;
    // 2. scaling, start
    hipLaunchKernelGGL(root_setup_kernel, dim3(ctl_blocks), dim3(128), 0, stream, d_fd, d_fs, d_state, cnt,
                       mode == ASTERIA_EPS_RELATIVE ? 1 : 0, pl.margin, root, pl.adapted ? 1 : 0);
    if (j64 > 0)
        hipLaunchKernelGGL(root_init_kernel<double>, dim3(tri_total), dim3(256), 0, stream, d_fd, d_fs, d_state,
                           cnt, tri_total, root);
    else
        hipLaunchKernelGGL(root_init_kernel<float>, dim3(tri_total), dim3(256), 0, stream, d_fd, d_fs, d_state,
                           cnt, tri_total, root);
    ASTERIA_HIP_TRY(hipGetLastError());

    // 3. coupled iteration
    for (int k = 0; k < K; ++k) {
        const bool p32 = k >= j64;
        hipLaunchKernelGGL(root_control_kernel, dim3(cnt), dim3(64), 0, stream, d_fd, d_fs, d_state, k,
                           p32 ? 1 : 0, 0, pl.stop_resid, root, pl.adapted ? 1 : 0, pl.xt_lowp ? 1 : 0);
        const int pa = k & 1;
        const bool lowp = p32 && k >= jlow;
        // X' = X T (X_1 comes from the start kernel).  X only needs the accuracy of the result, so
        // the update runs on the fp16 cores with split operands (22 bits) whenever the low-precision
        // tier is chosen automatically, from the first product on; otherwise with the tier of M.
        if (k > 0) {
            if (pl.xt_lowp || lowp)
                ASTERIA_HIP_TRY((launch_gemm_bf16_grouped<float, float, 2, 2, true, false>(d_xt[pa], cnt, tri_total, d_state, stream)));
            else
                ASTERIA_HIP_TRY((launch_gemm_grouped<float, float, float, false, false>(d_xt[pa], cnt, tri_total, d_state, stream)));
        }
        if (lowp) {
            ASTERIA_HIP_TRY((launch_gemm_bf16_grouped<float, float, 2, 2, true, false>(d_tab[0][pa][0], cnt, tri_total, d_state, stream)));
            if (root == 4)
                ASTERIA_HIP_TRY((launch_gemm_bf16_grouped<float, float, 2, 2, true, false>(d_tab[0][pa][1], cnt, tri_total, d_state, stream)));
            ASTERIA_HIP_TRY((launch_gemm_bf16_grouped<float, float, 2, 2, true, false>(d_tab[0][pa][2], cnt, tri_total, d_state, stream)));
        } else if (p32) {
            ASTERIA_HIP_TRY((launch_gemm_grouped<float, float, float, false, false>(d_tab[0][pa][0], cnt, tri_total, d_state, stream)));
            if (root == 4)
                ASTERIA_HIP_TRY((launch_gemm_grouped<float, float, float, false, false>(d_tab[0][pa][1], cnt, tri_total, d_state, stream)));
            ASTERIA_HIP_TRY((launch_gemm_grouped<float, float, float, false, false>(d_tab[0][pa][2], cnt, tri_total, d_state, stream)));
        } else {
            for (int l = 0; l < 3; ++l) {
                if (l == 1 && root != 4) continue;
                // the M-update of the last fp64 iteration writes the fp32 M the next tier starts from
                const GemmProblem *tab = (l == 2 && k == j64 - 1 && pl.use32) ? d_last64[pa] : d_tab[1][pa][l];
                if (ns8 > 0) {
                    // Cut the A operand into slices, decide per factor, multiply.  T goes to buffer 1
                    // and stays there: T T reads it twice, and T^4 M reads it as M (B mode 1), so M
                    // itself is never cut; T^2 and T^4 go to buffer 0.
                    const dim3 sgrid((unsigned)((i8_rows(n_max) + 3) / 4), (unsigned)cnt);
                    const int abuf = l == 0 ? 1 : 0, bbuf = l == 1 ? 0 : 1, bmode = l == 2 ? 1 : 0;
                    const int lds_k = i8_slice_lds_k(n_max);
                    {   // rows of 1900 to 2048 entries park more than the default 64 KiB of dynamic LDS
                        static bool cfg5s[MAX_DEVICES] = {}, cfg4s[MAX_DEVICES] = {};
                        if (ns8 == 5) ASTERIA_HIP_TRY(ensure_dynamic_lds(reinterpret_cast<const void *>(i8_slice_kernel<5>), i8_slice_lds_bytes(I8_SLICE_LDS_K), cfg5s));
                        else ASTERIA_HIP_TRY(ensure_dynamic_lds(reinterpret_cast<const void *>(i8_slice_kernel<4>), i8_slice_lds_bytes(I8_SLICE_LDS_K), cfg4s));
                    }
                    if (ns8 == 5) hipLaunchKernelGGL(i8_slice_kernel<5>, sgrid, dim3(256), i8_slice_lds_bytes(lds_k), stream, tab, d_xf, d_state, 0, abuf, lds_k);
                    else hipLaunchKernelGGL(i8_slice_kernel<4>, sgrid, dim3(256), i8_slice_lds_bytes(lds_k), stream, tab, d_xf, d_state, 0, abuf, lds_k);
                    // per factor: 4 slices where the estimate allows, else 5 (if the planes have them), else fp64
                    hipLaunchKernelGGL(i8_gate_kernel, dim3(ctl_blocks), dim3(128), 0, stream, d_xf, cnt, &d_fs[0].lo_cur,
                                       (int)sizeof(FactorScal), 4, ns8, abuf, bbuf, bmode,
                                       I8_THETA * 2.0f / (float)std::max(2, j64), d_state, profile_i8_counters());
                    ASTERIA_HIP_TRY(hipGetLastError());
                    if (ns8 == 5) ASTERIA_HIP_TRY((launch_gemm_i8_grouped<5>(tab, d_xf, cnt, tri_total, d_state, abuf, bbuf, bmode, stream)));
                    else ASTERIA_HIP_TRY((launch_gemm_i8_grouped<4>(tab, d_xf, cnt, tri_total, d_state, abuf, bbuf, bmode, stream)));
                }
                ASTERIA_HIP_TRY((launch_gemm_grouped<double, double, double, false, false>(tab, cnt, tri_total, d_state, stream)));
            }
        }
    }
    hipLaunchKernelGGL(root_control_kernel, dim3(cnt), dim3(64), 0, stream, d_fd, d_fs, d_state, K,
                       (K >= j64 && pl.use32) ? 1 : 0, 1, pl.stop_resid, root, pl.adapted ? 1 : 0, pl.xt_lowp ? 1 : 0);
    hipLaunchKernelGGL(root_finalize_kernel, dim3(sq_total), dim3(256), 0, stream, d_fd, d_fs, d_state, cnt,
                       d_sq, first, info, iters, resid, lambda_max);
    ASTERIA_HIP_TRY(hipGetLastError());
    return ASTERIA_OK;
}

// Which path a call takes and the workspace its factors need.  A call is accepted where its largest factor fits
// the workspace on the fp32 / fp64 path; the plane path is taken where that factor fits it too.
struct PassBytes {
    const Plan &pl;
    bool planes = false, f64 = false, fits = true;
    PassBytes(const asteria_factor *f, int nf, asteria_eps_mode mode, const float *eps, int eps_count, const Plan &p, size_t ws_bytes) : pl(p)
    {
        int n_max = 0;
        for (int i = 0; i < nf; ++i) n_max = std::max(n_max, f[i].n);
        double a_min = 1.0;
        for (int i = 0; i < eps_count; ++i) a_min = std::min(a_min, (double)eps[i] / (1.0 + (double)pl.margin + (double)eps[i]));
        fits = fixed_bytes() + of(n_max) <= ws_bytes;
        planes = plane_path(pl, mode, n_max);
        f64 = planes && plane_needs_f64(pl, 0.5 * a_min, n_max);
        if (planes && fixed_bytes() + of(n_max) > ws_bytes) planes = f64 = false;
    }
    size_t of(int n) const
    {
        return factor_small_bytes(n) + (planes ? plane_factor_bytes(n, pl.fp64_iters > 0, f64)
                                               : factor_table_bytes(n) + factor_matrix_bytes(n, pl.use64, pl.use32) + factor_i8_bytes(n, pl.i8_slices));
    }
};

}  // namespace

extern "C" asteria_status asteria_inverse_root_plan(int root, asteria_eps_mode mode, const float *eps, int eps_count,
                                                    const asteria_root_opts *opts, int32_t *fp64_iters,
                                                    int32_t *lowp_from, int32_t *x_update_lowp)
{
    if (root != 2 && root != 4) return ASTERIA_UNSUPPORTED;
    if (!eps || eps_count <= 0) return ASTERIA_INVALID_ARG;
    Plan pl;
    const asteria_status st = make_plan(opts, mode, eps, eps_count, root, pl);
    if (st != ASTERIA_OK) return st;
    if (fp64_iters) *fp64_iters = pl.fp64_iters;
    if (lowp_from) *lowp_from = pl.lowp_from;
    if (x_update_lowp) *x_update_lowp = pl.xt_lowp ? 1 : 0;
    return ASTERIA_OK;
}

extern "C" size_t asteria_inverse_root_workspace_bytes(const asteria_factor *f, int nfactors,
                                                       const asteria_root_opts *opts, size_t *min_bytes)
{
    if (min_bytes) *min_bytes = 0;
    if (!f || nfactors <= 0) return 0;
    Plan pl;
    const float e1 = 1e-6f;
    if (make_plan(opts, ASTERIA_EPS_RELATIVE, &e1, 1, 4, pl) != ASTERIA_OK) return 0;
    // sizes must not depend on eps: reserve both precisions unless the caller pinned one
    asteria_root_opts o;
    asteria_root_opts_default(&o);
    if (opts) o = *opts;
    const bool use64 = (o.fp64_iters != 0);
    const bool use32 = !(o.fp64_iters >= o.max_iters && o.fp64_iters > 0);
    size_t total = fixed_bytes(), biggest = 0;
    for (int i = 0; i < nfactors; ++i) {
        if (f[i].n <= 0) return 0;
        // the call takes one of two paths (eps and root decide; pinned precision options never the second): room for either
        size_t b = factor_table_bytes(f[i].n) + factor_matrix_bytes(f[i].n, use64, use32) +
                   factor_i8_bytes(f[i].n, use64 ? (o.int8_slices < 0 ? 5 : o.int8_slices) : 0);
        if (o.fp64_iters < 0 && o.lowp_from < 0) b = std::max(b, plane_factor_bytes(f[i].n, true, true));
        b += factor_small_bytes(f[i].n);
        total += b;
        biggest = std::max(biggest, b);
    }
    if (min_bytes) *min_bytes = biggest + fixed_bytes();
    return total;
}

namespace {
asteria_status inverse_root(const asteria_factor *f, int nfactors, int root, asteria_eps_mode mode, const float *eps, int eps_count,
                            const asteria_root_opts *opts, int32_t *info, int32_t *iters, float *resid, float *lambda_max,
                            void *ws, size_t ws_bytes, void *stream_, LanczosWaits waits)
{
    asteria_status st = validate(f, nfactors, root, eps, eps_count);
    if (st != ASTERIA_OK) return st;
    if (mode != ASTERIA_EPS_RELATIVE && mode != ASTERIA_EPS_ABSOLUTE) return ASTERIA_INVALID_ARG;
    Plan pl;
    st = make_plan(opts, mode, eps, eps_count, root, pl);
    if (st != ASTERIA_OK) return st;
    pl.waits = waits;
    if (!ws) return ASTERIA_WORKSPACE_TOO_SMALL;
    if (reinterpret_cast<uintptr_t>(ws) & 255u) return ASTERIA_INVALID_ARG;   // workspace must be 256-byte aligned
    hipStream_t stream = reinterpret_cast<hipStream_t>(stream_);

    // Passes cover contiguous index ranges of the caller's order (outputs are indexed by caller position), each the
    // largest that fits the workspace.
    const PassBytes pb(f, nfactors, mode, eps, eps_count, pl, ws_bytes);
    if (!pb.fits) return ASTERIA_WORKSPACE_TOO_SMALL;
    int first = 0;
    while (first < nfactors) {
        size_t used = fixed_bytes();
        int cnt = 0;
        while (first + cnt < nfactors && cnt < 65535) {   // 65535: y extent of the mat-vec grid
            const size_t b = pb.of(f[first + cnt].n);
            if (used + b > ws_bytes) break;
            used += b;
            ++cnt;
        }
        if (cnt == 0) return ASTERIA_WORKSPACE_TOO_SMALL;
        if (pb.planes) st = run_pass_planes(f, first, cnt, eps, eps_count, pl, pb.f64, info, iters, resid, lambda_max, ws, stream);
        else st = run_pass(f, first, cnt, root, mode, eps, eps_count, pl, info, iters, resid, lambda_max, ws, stream);
        if (st != ASTERIA_OK) return st;
        first += cnt;
    }
    return ASTERIA_OK;
}
}  // namespace

extern "C" asteria_status asteria_inverse_root(const asteria_factor *f, int nfactors, int root,
                                               asteria_eps_mode mode, const float *eps, int eps_count,
                                               const asteria_root_opts *opts,
                                               int32_t *info, int32_t *iters, float *resid, float *lambda_max,
                                               void *ws, size_t ws_bytes, void *stream)
{
    return inverse_root(f, nfactors, root, mode, eps, eps_count, opts, info, iters, resid, lambda_max, ws, ws_bytes, stream, LanczosWaits{});
}

extern "C" asteria_status asteria_inverse_root_waits(const asteria_factor *f, int nfactors, int root,
                                                     asteria_eps_mode mode, const float *eps, int eps_count,
                                                     const asteria_root_opts *opts,
                                                     int32_t *info, int32_t *iters, float *resid, float *lambda_max,
                                                     void *ws, size_t ws_bytes, void *stream, uint32_t looks_sums, uint32_t looks_y)
{
    return inverse_root(f, nfactors, root, mode, eps, eps_count, opts, info, iters, resid, lambda_max, ws, ws_bytes, stream,
                        LanczosWaits{looks_sums, looks_y});
}

// ---- the same call for callers that cannot allocate ---------------------------------------------
// The workspace is a fixed array in the library's device image instead of caller memory.  In host
// code the array's name only stands for the symbol: its device address is looked up once per device
// and that pointer is what the kernels (and nothing else here) receive.
namespace {
constexpr size_t STATIC_SCRATCH_BYTES = (size_t)64 << 20;
constexpr int STATIC_SCRATCH_MAX_DEVICES = 64;
}  // namespace
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];
static void *g_scratch_ptr[STATIC_SCRATCH_MAX_DEVICES];   // device address of `scratch`, per device

extern "C" size_t asteria_static_scratch_bytes(void) { return STATIC_SCRATCH_BYTES; }

extern "C" asteria_status asteria_inverse_root_static(const asteria_factor *f, int nfactors, int root,
                                                      asteria_eps_mode mode, const float *eps, int eps_count,
                                                      const asteria_root_opts *opts,
                                                      int32_t *info, int32_t *iters, float *resid, float *lambda_max,
                                                      void *stream_)
{
    asteria_status st = validate(f, nfactors, root, eps, eps_count);
    if (st != ASTERIA_OK) return st;
    if (mode != ASTERIA_EPS_RELATIVE && mode != ASTERIA_EPS_ABSOLUTE) return ASTERIA_INVALID_ARG;
    Plan pl;
    st = make_plan(opts, mode, eps, eps_count, root, pl);
    if (st != ASTERIA_OK) return st;
    // every factor must fit the array by itself (the call works through the batch in passes)
    if (!PassBytes(f, nfactors, mode, eps, eps_count, pl, STATIC_SCRATCH_BYTES).fits) return ASTERIA_EXCEEDS_STATIC_SCRATCH;
    int dev = -1;
    ASTERIA_HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= STATIC_SCRATCH_MAX_DEVICES) return ASTERIA_UNSUPPORTED;
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        ASTERIA_HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return ASTERIA_HIP_ERROR;
        g_scratch_ptr[dev] = p;
    }
    return asteria_inverse_root(f, nfactors, root, mode, eps, eps_count, opts, info, iters, resid, lambda_max,
                                g_scratch_ptr[dev], STATIC_SCRATCH_BYTES, stream_);
}
