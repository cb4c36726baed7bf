// lambda_max of every factor by a Lanczos process.
//
// v_0 a fixed pseudo-random vector; step j: y = A v_j, alpha_j = v_j^T y, w = y - alpha_j v_j - beta_{j-1} v_{j-1},
// beta_j = ||w||, v_{j+1} = w / beta_j.  The estimate is the largest eigenvalue of the tridiagonal matrix
// (alpha, beta) of the steps so far: it rises monotonically to lambda_max and gets there in about 1 / sqrt(gap)
// steps where plain power iteration needs 1 / gap.  No re-orthogonalisation: what fp32 round-off does to the
// later vectors produces copies of converged Ritz values, never one above lambda_max by more than round-off.
// A factor stops once three consecutive steps have raised the estimate by less than tol2 of it, or where the
// recurrence ends (beta = 0, an invariant subspace: the estimate is exact).
//
// Who computes a step:
//   lanczos_factor_kernel   one workgroup per factor takes all steps in one launch: n <= 256 with the matrix in
//                           registers, larger ones streamed.  For small factors, and for batches that keep every
//                           CU busy anyway.
//   lanczos_cluster_kernel  several workgroups per factor, the matrix in their registers, all steps in one launch: n <= 2048
//   lanczos_step_kernel     one launch per step, a factor's rows spread over workgroups: few large factors.  Every
//                           workgroup forms the next vector by itself from the previous step's y (n elements, against
//                           n rows of n), so a step is one launch; an extra workgroup keeps the recurrence.
//   pm_packed_* + pm_lanczos_kernel  large factors in packed lower tiles: every stored tile is read once.
#pragma once
#include "gemm.h"
#include "root_factor.h"

namespace asteria {

constexpr int LZ_ROWS = 32;      // rows of A per workgroup of lanczos_step_kernel
// figures beside lanczos_by_factor
constexpr int LZ_WG_N = 512;     // largest n that lanczos_factor_kernel takes in any batch
constexpr int LZ_WG_BATCH = 192; // it takes every n where the batch has as many elements as this number of its largest factors
constexpr int LZ_WG_MAX_N = 8192;   // its vectors fit LDS

__device__ __forceinline__ float hash_unit(uint32_t f, uint32_t j)
{
    uint32_t x = j * 0x9E3779B1u + f * 0x85EBCA77u + 0x165667B1u;
    x ^= x >> 15; x *= 0x2C1B3C6Du; x ^= x >> 12; x *= 0x297A2D39u; x ^= x >> 15;
    return (float)(x >> 8) * (1.0f / 8388608.0f) - 1.0f;   // [-1, 1)
}

__device__ __forceinline__ double square_sum(const float4 &t)
{
    return (double)t.x * (double)t.x + (double)t.y * (double)t.y + (double)t.z * (double)t.z + (double)t.w * (double)t.w;
}

// One wavefront: largest eigenvalue of the symmetric tridiagonal matrix with diagonal a[0 .. m) and off-diagonal
// b[0 .. m - 1), given `before`, that of the leading m - 1 rows (ignored for m = 1).  It lies in
// [max(before, a_m), max(before, a_m) + |b_{m-1}|]; every lane tests one point of the bracket (all leading minors
// of x I - T positive, by the three-term recurrence of the characteristic polynomials).  The first round's points lie
// in powers of 1.38 from the lower end, 9 decades of what the last step may have raised the value by; every further round narrows
// the bracket 65-fold: 2 to 4 rounds to 1e-8.
// a, b: 16-byte aligned arrays of LZ_MAX in LDS, read eight rows at a time (what lies beyond row m is not used).
__device__ inline double tridiag_largest(const float *a, const float *b, int m, double before)
{
    const int lane = threadIdx.x & 63;
    if (m == 1) return (double)a[0];
    double lo = fmax(before, (double)a[m - 1]), hi = lo + fabs((double)b[m - 2]);
    if (!(hi > lo) || !(hi < 1e300) || !(hi > 0.0)) return lo;
    hi += 1e-9 * hi;
    const double inv = 1.0 / hi;
    for (int round = 0; round < 7 && hi - lo > 1e-8 * hi; ++round) {
        auto share = [&](int i) __attribute__((always_inline)) {
            return round == 0 ? (double)exp2f(-0.46875f * (float)(63 - i)) : (double)(i + 1) * (1.0 / 65.0);
        };
        const double w = hi - lo, x = lo + w * share(lane), xs = x * inv;
        double p = 1.0, q = 0.0, b2 = 0.0;             // minors of x I - T, of order i and i - 1
        bool above = true;
        for (int i0 = 0; i0 < m; i0 += 8) {
            float4 va[2], vb[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                va[e] = *reinterpret_cast<const float4 *>(a + i0 + 4 * e);
                vb[e] = *reinterpret_cast<const float4 *>(b + i0 + 4 * e);
            }
            const float ra[8] = {va[0].x, va[0].y, va[0].z, va[0].w, va[1].x, va[1].y, va[1].z, va[1].w};
            const float rb[8] = {vb[0].x, vb[0].y, vb[0].z, vb[0].w, vb[1].x, vb[1].y, vb[1].z, vb[1].w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                // rows beyond the last leave the minor as it is
                const double t = (i0 + e < m ? xs - (double)ra[e] * inv : 1.0) * p - (i0 + e < m ? b2 : 0.0) * q;
                q = p; p = t;
                above = above && p > 0.0;
                const double bi = (double)rb[e] * inv;
                b2 = bi * bi;
            }
            if (fabs(p) < 1e-60 && fabs(q) < 1e-60) { p *= 1e60; q *= 1e60; }
        }
        const uint64_t mask = __ballot(above);
        const int first = mask ? __ffsll((long long)mask) - 1 : 64;     // first point at or above the largest eigenvalue
        if (first < 64) hi = lo + w * share(first);
        if (first > 0) lo = lo + w * share(first - 1);
    }
    return 0.5 * (lo + hi);
}

// After step j: a, b hold the recurrence up to alpha_j, beta_j (in LDS: every lane walks through it).  One
// wavefront; rho, small: the estimate and how many steps have not moved it.  Returns whether the factor is finished.
__device__ inline bool lanczos_advance(float &rho, int &small, const float *a, const float *b, int j, float beta, float tol2)
{
    const double before = j > 0 ? (double)rho : 0.0;
    const double theta = tridiag_largest(a, b, j + 1, before);
    const bool ended = !(beta > 1e-7f * fabsf((float)theta)) || !(beta > 0.0f);
    small = (j > 0 && theta - before <= (double)tol2 * fabs(theta)) ? small + 1 : 0;
    rho = (float)theta;
    return ended || small >= 3;
}
// ... with both kept in the factor's state
__device__ inline bool lanczos_advance(FactorScal &S, const float *a, const float *b, int j, float beta, float tol2)
{
    float rho = S.rho;
    int small = S.lz_small;
    const bool end = lanczos_advance(rho, small, a, b, j, beta, tol2);
    if ((threadIdx.x & 63) == 0) { S.rho = rho; S.lz_small = small; }
    return end;
}

// ---- one workgroup per factor --------------------------------------------------------------------------
constexpr int LZ_THREADS = 1024, LZ_FEW_THREADS = 512, LZ_FEW_N = 128;

__device__ __forceinline__ float row_sum16(float v)       // sum over 16 consecutive lanes
{
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// RESIDENT: every factor has n <= 256 and is held in registers; on 512 threads where all have n <= 128 (the same sums in the same order,
// fewer wavefronts to wait for at a barrier; refresh of one factor of 128 and one of 100 274 -> 264 us, of 600 of n = 128 1380 -> 1332).  resume >= 0: continue after that many launches
// of lanczos_step_kernel.
template <bool RESIDENT, int THREADS = LZ_THREADS>
__global__ __launch_bounds__(THREADS) void lanczos_factor_kernel(const FactorDev *fd, FactorScal *fs, float tol2, int steps, int resume, int ld)
{
    constexpr int WAVES = THREADS / 64, NI = THREADS == LZ_FEW_THREADS ? 2 : 4;     // NI: of 64 columns each
    const int f = blockIdx.x;
    FactorScal &S = fs[f];
    if (resume >= 0 && S.pm_done) return;
    const FactorDev &F = fd[f];
    const int n = F.n, lda = F.ldw;
    const float *__restrict__ A = F.Aw;
    extern __shared__ __align__(16) float lz_smem[];
    float *v = lz_smem, *vp = v + ld, *y = vp + ld;          // ld: n of the largest factor, padded to 256
    __shared__ float red[WAVES];
    __shared__ double redd[2][WAVES];
    __shared__ __align__(16) float la[LZ_MAX], lb[LZ_MAX];
    __shared__ int done;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool vec = ((reinterpret_cast<uintptr_t>(A) & 15u) == 0) && ((lda & 3) == 0);
    auto block_sum = [&](double x) -> double {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
        __syncthreads();
        if (lane == 0) redd[0][wave] = x;
        __syncthreads();
        double t = 0.0;
        for (int w = 0; w < WAVES; ++w) t += redd[0][w];
        return t;
    };
    // n <= 256: lane group g of 16 in wavefront w holds rows 16 w + 4 g .. + 3, lane c of it the columns 4 (c + 16 i) .. + 3
    float ar[RESIDENT ? 4 : 1][4 * NI];
    const int rg = 16 * wave + 4 * (lane >> 4), cl = lane & 15;
    if constexpr (RESIDENT) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int r = rg + q, c = 4 * (cl + 16 * i);
                if (vec && r < n && c + 4 <= n) {
                    const float4 t = *reinterpret_cast<const float4 *>(A + (size_t)r * lda + c);
                    ar[q][4 * i] = t.x; ar[q][4 * i + 1] = t.y; ar[q][4 * i + 2] = t.z; ar[q][4 * i + 3] = t.w;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) ar[q][4 * i + e] = (r < n && c + e < n) ? A[(size_t)r * lda + c + e] : 0.0f;
                }
            }
    }
    int j0 = 0;
    float beta_p = 0.0f;
    if (tid == 0) done = 0;
    if (resume < 0) {
        double s = 0.0;
        for (int i = tid; i < ld; i += THREADS) {
            // the same start vector for every factor: a factor's result does not depend on its place in the batch
            const float x = i < n ? hash_unit(0u, (uint32_t)i) : 0.0f;
            v[i] = x; vp[i] = 0.0f;
            s += (double)x * (double)x;
        }
        s = block_sum(s);
        const float inv = s > 0.0 ? (float)(1.0 / sqrt(s)) : 0.0f;
        for (int i = tid; i < ld; i += THREADS) v[i] *= inv;
        double saa = 0.0, str = 0.0;
        if constexpr (RESIDENT) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int e = 0; e < 4 * NI; ++e) saa += (double)ar[q][e] * (double)ar[q][e];
        }
        for (int i = tid; i < n; i += THREADS) str += (double)A[(size_t)i * lda + i];
        saa = block_sum(saa);                                // streamed factors: gathered in the first product
        str = block_sum(str);
        if (tid == 0) { S.fro2 = saa; S.trace = str; S.rho = 0.0f; S.lz_small = 0; S.pm_done = 0; }
    } else {
        j0 = resume - 1;                                     // its y is there, its alpha is not
        for (int i = tid; i < ld; i += THREADS) {
            v[i] = i < n ? F.pv[j0 % 3][i] : 0.0f;
            vp[i] = (i < n && j0 > 0) ? F.pv[(j0 + 2) % 3][i] : 0.0f;
            y[i] = i < n ? F.py[j0 & 1][i] : 0.0f;
        }
        beta_p = j0 > 0 ? S.lz_b[j0 - 1] : 0.0f;
        if (tid < j0) { la[tid] = S.lz_a[tid]; lb[tid] = S.lz_b[tid]; }
    }
    __syncthreads();
    bool stop = false;                                       // wavefront 0: the recurrence so far has settled
    for (int j = j0; j < steps; ++j) {
        float yv = 0.0f;
        if (j == j0 && resume >= 0) {
            for (int i = tid; i < n; i += THREADS) yv += y[i] * v[i];
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) yv += __shfl_xor(yv, off, 64);
        } else if constexpr (RESIDENT) {
            float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            if (16 * wave < n) {
#pragma unroll
                for (int i = 0; i < NI; ++i) {
                    const float4 x = *reinterpret_cast<const float4 *>(v + 4 * (cl + 16 * i));
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        s[q] += ar[q][4 * i] * x.x + ar[q][4 * i + 1] * x.y + ar[q][4 * i + 2] * x.z + ar[q][4 * i + 3] * x.w;
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) s[q] = row_sum16(s[q]);
            if (cl == 0) {
#pragma unroll
                for (int q = 0; q < 4; ++q) { y[rg + q] = s[q]; yv += s[q] * v[rg + q]; }
            }
            yv += __shfl_xor(yv, 16, 64);
            yv += __shfl_xor(yv, 32, 64);
        } else {
            double saa = 0.0;
            auto product = [&](auto first) {
                for (int r0 = 4 * wave; r0 < n; r0 += 4 * WAVES) {
                    float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
                    double q[4] = {0.0, 0.0, 0.0, 0.0};
                    const float *ap[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) ap[e] = A + (size_t)min(r0 + e, n - 1) * lda;
                    int c0 = 0;
                    if (vec) {
                        const int n4 = n >> 2;
#pragma unroll 2
                        for (int c = lane; c < n4; c += 64) {
                            const float4 x = reinterpret_cast<const float4 *>(v)[c];
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const float4 t = reinterpret_cast<const float4 *>(ap[e])[c];
                                s[e] += t.x * x.x + t.y * x.y + t.z * x.z + t.w * x.w;
                                if constexpr (decltype(first)::value) q[e] += square_sum(t);
                            }
                        }
                        c0 = n4 << 2;
                    }
#pragma unroll 4
                    for (int c = c0 + lane; c < n; c += 64) {
                        const float x = v[c];
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float t = ap[e][c];
                            s[e] += t * x;
                            if constexpr (decltype(first)::value) q[e] += (double)t * (double)t;
                        }
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
#pragma unroll
                        for (int off = 32; off > 0; off >>= 1) s[e] += __shfl_xor(s[e], off, 64);
                        if (r0 + e < n) {
                            if (lane == 0) y[r0 + e] = s[e];
                            yv += s[e] * v[r0 + e];
                            if constexpr (decltype(first)::value) saa += q[e];
                        }
                    }
                }
            };
            if (j == 0) {
                product(std::true_type{});
                saa = block_sum(saa);
                if (tid == 0) S.fro2 = saa;
            } else product(std::false_type{});
        }
        if (lane == 0) red[wave] = yv;
        if (tid == 0 && stop) done = 1;
        __syncthreads();
        if (done) break;
        double alpha_d = 0.0;
        for (int w = 0; w < WAVES; ++w) alpha_d += (double)red[w];
        const float alpha = (float)alpha_d;
        double ww = 0.0;
        for (int i = tid; i < n; i += THREADS) {
            const float x = y[i] - alpha * v[i] - beta_p * vp[i];
            y[i] = x;
            ww += (double)x * (double)x;
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) ww += __shfl_xor(ww, off, 64);
        if (lane == 0) redd[1][wave] = ww;
        __syncthreads();
        double ww_d = 0.0;
        for (int w = 0; w < WAVES; ++w) ww_d += redd[1][w];
        const float beta = (float)sqrt(ww_d);
        if (!(beta < 3.0e38f) || !(fabsf(alpha) < 3.0e38f)) {         // non-finite input (uniform)
            if (tid == 0) S.rho = NAN;
            break;
        }
        const float inv = beta > 0.0f ? 1.0f / beta : 0.0f;
        for (int i = tid; i < n; i += THREADS) {
            const float t = v[i];
            v[i] = y[i] * inv;
            vp[i] = t;
        }
        beta_p = beta;
        if (tid == 0) { la[j] = alpha; lb[j] = beta; }
        __syncthreads();
        // the recurrence is looked at by one wavefront while the others go on to the next product: they stop one
        // step later than they could
        if (wave == 0) stop = lanczos_advance(S, la, lb, j, beta, tol2);
    }
    if (tid == 0) S.pm_done = 1;
}

// ---- the matrix in the registers of several workgroups ---------------------------------------------------
// A factor's rows are dealt to lanczos_members(n) workgroups, which load them once and keep them; a step then moves n words per
// workgroup through memory instead of the matrix.  Every member forms alpha, beta and the next vector from all of y by itself, in the
// same order and so with the same bits: they agree on when to stop, and a step needs one exchange.
//
// The exchange: word i of a step holds y_i and the step's number in 64 bits, written and read by relaxed atomics of device scope, which
// carry their own validity: no fence (which would write back the whole L2: a phase of 72 workgroups took 6 us with it) and no flag.  Two
// buffers in turn: whoever writes step j + 2 has read all of step j + 1, which nobody publishes before having read step j.
//
// Progress: a workgroup takes its (factor, member) by a ticket, so whoever waits waits for the holders of tickets next to its own;
// unfinished factors below the last ticket taken have all their members on the chip, and the one at the frontier, with at most
// lanczos_members(2048) = 43, finds room as soon as those below are done.  That room may be taken: by a mask of the stream's CUs, by kernels
// of other processes that do not end.  So both waits, of the first member for the others' sums and of every member for y, are bounded, and a
// member that gives up sets a word for the launch that ends all waits in it.  A factor whose first member has not settled is left to
// lanczos_alone, one workgroup that waits for nobody.
//
// Bound by the first load (HBM) and by a step's chain: exchange, two block sums, the product, the tridiagonal problem, which grows with the
// steps.  n = 257 .. 1500, evenly spaced spectrum: 8 us from the 8th to the 16th step, 9 to the 24th, 10 to the 48th; n = 2048 10 - 13.
// 168 registers are all that 12 wavefronts leave each other; with 128 for the matrix 168 values spill (148 bytes of scratch a
// lane, written once and read in part in every step): the estimate of the 1.1B model, 7.1 ms, moves 10.8 GB in and 1.8 out where the
// matrices are 7.2 (mean of full and packed).  Whole refreshes beside lanczos_by_cluster.
constexpr uint32_t LC_POLLS = 1u << 21;
struct LanczosWaits { uint32_t sums = LC_POLLS, y = LC_POLLS; };      // looks at what others have to write before a member gives up

__device__ __forceinline__ void word_put(ASTERIA_GLOBAL uint64_t *p, uint32_t value, uint32_t tag)
{
    __hip_atomic_store(p, (uint64_t)value | ((uint64_t)tag << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t word_get(const ASTERIA_GLOBAL uint64_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Exchange words of every factor to zero (no step's number), its members into the map, the ticket and the word of a wait given up to zero.
__global__ __launch_bounds__(256) void lanczos_prepare_kernel(const FactorDev *fd, FactorScal *fs, uint2 *map, int *ticket)
{
    const FactorDev &F = fd[blockIdx.x];
    const int words = (int)lanczos_words(F.n), members = lanczos_members(F.n);
    for (int i = threadIdx.x; i < words; i += 256) F.lz_words[i] = 0;
    for (int m = threadIdx.x; m < members; m += 256) map[F.lz_start + m] = make_uint2(blockIdx.x, (unsigned)m);
    if (threadIdx.x == 0) fs[blockIdx.x].pm_done = 0;
    if (blockIdx.x == 0 && threadIdx.x < 2) ticket[threadIdx.x] = 0;
}

// NI: a lane holds columns 4 lane + 256 i .. + 3 for i < NI of RW consecutive rows (128 values)
template <int NI>
__device__ __forceinline__ void lanczos_member(const FactorDev &F, FactorScal &S, int member, float tol2, int steps, LanczosWaits waits, int *given_up)
{
    constexpr int RW = 32 / NI, RB = RW < 8 ? RW : 8, OWN = (256 * NI + LC_THREADS - 1) / LC_THREADS;
    __shared__ __align__(16) float v_lds[256 * NI];
    __shared__ double redd[2][LC_WAVES];
    __shared__ __align__(16) float la[LZ_MAX], lb[LZ_MAX];
    __shared__ int done, gave_up;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = F.n, members = lanczos_members(n), row0 = member * LC_WAVES * RW + wave * RW;
    ASTERIA_GLOBAL uint64_t *words = (ASTERIA_GLOBAL uint64_t *)F.lz_words, *sums = words + 2 * (size_t)n;
    float ar[RW][4 * NI];
    if (!F.a_packed) {
        // No branches between the loads and no masks: addresses are kept inside the matrix.  What a row beyond it gives is not written,
        // a column beyond it meets a zero of v
        typedef float floatx4_any __attribute__((ext_vector_type(4), aligned(4)));
        const ASTERIA_GLOBAL float *A = (const ASTERIA_GLOBAL float *)F.A;
        const int lda = F.lda, n4 = n & ~3;
        if (n4 > 0) {
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int q = 0; q < RW; ++q) {
                    const floatx4_any t = *(const ASTERIA_GLOBAL floatx4_any *)(A + (size_t)min(row0 + q, n - 1) * lda + min(4 * lane + 256 * i, n4 - 4));
#pragma unroll
                    for (int e = 0; e < 4; ++e) ar[q][4 * i + e] = t[e];
                }
        } else {
#pragma unroll
            for (int q = 0; q < RW; ++q)
#pragma unroll
                for (int e = 0; e < 4 * NI; ++e) ar[q][e] = 0.0f;
        }
        if (n4 != n)
#pragma unroll
            for (int i = 0; i < NI; ++i)
                if (n4 / 256 == i && 4 * lane + 256 * i == n4)
#pragma unroll
                    for (int q = 0; q < RW; ++q)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            ar[q][4 * i + e] = n4 + e < n ? A[(size_t)min(row0 + q, n - 1) * lda + n4 + e] : 0.0f;
    } else {
        // packed tiles are whole: their padding is read and masked.  Above the diagonal: column c of these rows is row c of the mirror tile
        const int ti = row0 / PACK_T, rt = row0 % PACK_T;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int c = 4 * lane + 256 * i, tj = c / PACK_T, ct = c % PACK_T;
            const bool some = row0 < n && c < n, below = tj <= ti;
            if (some && below) {
                const ASTERIA_GLOBAL float *t = (const ASTERIA_GLOBAL float *)F.A + ((size_t)(ti * (ti + 1) / 2 + tj) * PACK_T + rt) * PACK_T + ct;
#pragma unroll
                for (int q = 0; q < RW; ++q) {
                    const floatx4 x = *(const ASTERIA_GLOBAL floatx4 *)(t + (size_t)q * PACK_T);
                    ar[q][4 * i] = x[0]; ar[q][4 * i + 1] = x[1]; ar[q][4 * i + 2] = x[2]; ar[q][4 * i + 3] = x[3];
                }
            } else if (some) {
                const ASTERIA_GLOBAL float *t = (const ASTERIA_GLOBAL float *)F.A + ((size_t)(tj * (tj + 1) / 2 + ti) * PACK_T + ct) * PACK_T + rt;
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int q = 0; q < RW; q += 4) {
                        const floatx4 x = *(const ASTERIA_GLOBAL floatx4 *)(t + (size_t)e * PACK_T + q);
                        ar[q][4 * i + e] = x[0]; ar[q + 1][4 * i + e] = x[1]; ar[q + 2][4 * i + e] = x[2]; ar[q + 3][4 * i + e] = x[3];
                    }
            }
#pragma unroll
            for (int q = 0; q < RW; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (row0 + q >= n || c + e >= n) ar[q][4 * i + e] = 0.0f;
        }
    }
    auto wave_sum = [](double x) __attribute__((always_inline)) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
        return x;
    };
    auto block_sum = [&](double x, double *red) __attribute__((always_inline)) {     // ends with red full and a barrier passed
        x = wave_sum(x);
        if (lane == 0) red[wave] = x;
        __syncthreads();
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < LC_WAVES; ++w) t += red[w];
        return t;
    };
    // the vectors: elements tid + 768 q in registers, v in LDS as well
    float v[OWN], vp[OWN];
    double ss = 0.0;
#pragma unroll
    for (int q = 0; q < OWN; ++q) {
        const int i = tid + LC_THREADS * q;
        // the same start vector for every factor: a factor's result does not depend on its place in the batch
        v[q] = i < n ? hash_unit(0u, (uint32_t)i) : 0.0f;
        vp[q] = 0.0f;
        ss += (double)v[q] * (double)v[q];
    }
    if (tid == 0) done = gave_up = 0;
    ss = block_sum(ss, redd[0]);
    const float inv0 = ss > 0.0 ? (float)(1.0 / sqrt(ss)) : 0.0f;
    bool lost = false;                                       // this wavefront gave up a wait
    // every 64th look: somebody gave up
    auto hopeless = [&](uint32_t looks) __attribute__((always_inline)) {
        return (looks & 63u) == 63u && __hip_atomic_load(given_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
    };
#pragma unroll
    for (int q = 0; q < OWN; ++q) {
        const int i = tid + LC_THREADS * q;
        v[q] *= inv0;
        if (i < 256 * NI) v_lds[i] = v[q];
    }
    {
        // ||A||_F^2 and the trace: of this member's rows, collected by the first member
        double saa = 0.0, str = 0.0;
#pragma unroll
        for (int q = 0; q < RW; ++q)
#pragma unroll
            for (int e = 0; e < 4 * NI; ++e) {
                const float x = row0 + q < n && 4 * lane + 64 * (e & ~3) < n ? ar[q][e] : 0.0f;
                saa += (double)x * (double)x;
            }
        if (lane < RW && row0 + lane < n) {
            const int r = row0 + lane;
            str = (double)F.A[F.a_packed ? packed_off(r, r) : (size_t)r * F.lda + r];
        }
        saa = block_sum(saa, redd[1]);
        __syncthreads();
        str = block_sum(str, redd[0]);
        if (tid == 0 && members > 1) {
            const uint64_t a = (uint64_t)__double_as_longlong(saa), t = (uint64_t)__double_as_longlong(str);
            ASTERIA_GLOBAL uint64_t *d = sums + 4 * (size_t)member;
            word_put(d, (uint32_t)a, 1u); word_put(d + 1, (uint32_t)(a >> 32), 1u);
            word_put(d + 2, (uint32_t)t, 1u); word_put(d + 3, (uint32_t)(t >> 32), 1u);
        }
        if (member == 0 && members > 1) {
            // (43 members at most: one lane each)
            double a = 0.0, t = 0.0;
            if (wave == 0) {
                bool all = lane >= members;
                if (!all) {
                    const ASTERIA_GLOBAL uint64_t *d = sums + 4 * (size_t)lane;
                    uint64_t w[4] = {0, 0, 0, 0};
                    for (uint32_t p = 0; p < waits.sums; ++p) {
                        all = true;
#pragma unroll
                        for (int e = 0; e < 4; ++e) { w[e] = word_get(d + e); all = all && (uint32_t)(w[e] >> 32) == 1u; }
                        if (all || hopeless(p)) break;
                        __builtin_amdgcn_s_sleep(1);
                    }
                    a = __longlong_as_double((long long)((w[0] & 0xffffffffull) | (w[1] << 32)));
                    t = __longlong_as_double((long long)((w[2] & 0xffffffffull) | (w[3] << 32)));
                }
                lost = !__all(all);
                a = wave_sum(a); t = wave_sum(t);
            }
            saa = a; str = t;
        }
        if (member == 0 && tid == 0) { S.fro2 = saa; S.trace = str; S.rho = 0.0f; S.lz_small = 0; }
    }
    __syncthreads();
    float beta_p = 0.0f, rho = 0.0f;
    int small = 0;
    bool stop = false, settled = true;
    for (int j = 0; j < steps; ++j) {
        // ---- this member's rows of y, RB at a time
#pragma unroll
        for (int b = 0; b < RW; b += RB) {
            float s[RB];
#pragma unroll
            for (int q = 0; q < RB; ++q) s[q] = 0.0f;
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const float4 x = *reinterpret_cast<const float4 *>(v_lds + 4 * lane + 256 * i);
#pragma unroll
                for (int q = 0; q < RB; ++q)
                    s[q] += ar[b + q][4 * i] * x.x + ar[b + q][4 * i + 1] * x.y + ar[b + q][4 * i + 2] * x.z + ar[b + q][4 * i + 3] * x.w;
            }
            // a level halves the rows a lane holds a part of
            int row = row0 + b, off = 32;
#pragma unroll
            for (int half = RB / 2; half > 0; half /= 2, off >>= 1) {
                const bool up = (lane & off) != 0;
#pragma unroll
                for (int q = 0; q < half; ++q) {
                    const float give = up ? s[q] : s[q + half], keep = up ? s[q + half] : s[q];
                    s[q] = keep + __shfl_xor(give, off, 64);
                }
                row += up ? half : 0;
            }
            const int others = lane & (2 * off - 1);
#pragma unroll
            for (; off > 0; off >>= 1) s[0] += __shfl_xor(s[0], off, 64);
            if (others == 0 && row < n) word_put(words + (size_t)(j & 1) * n + row, __float_as_uint(s[0]), (uint32_t)j + 1u);
        }
        if (tid == 0 && stop) done = 1;
        // ---- all of y
        float y[OWN];
        double yv = 0.0;
        {
            uint64_t w[OWN] = {};
            for (uint32_t polls = 0; !lost; ++polls) {
                if (polls == waits.y || __any(hopeless(polls))) { lost = true; break; }
                bool all = true;
#pragma unroll
                for (int q = 0; q < OWN; ++q) {
                    const int i = tid + LC_THREADS * q;
                    w[q] = i < n ? word_get(words + (size_t)(j & 1) * n + i) : (uint64_t)(j + 1) << 32;
                    all = all && (uint32_t)(w[q] >> 32) == (uint32_t)j + 1u;
                }
                if (__all(all)) break;
            }
#pragma unroll
            for (int q = 0; q < OWN; ++q) {
                y[q] = lost ? NAN : __uint_as_float((uint32_t)w[q]);
                yv += (double)(y[q] * v[q]);
            }
        }
        if (lost && lane == 0) {
            gave_up = 1;
            __hip_atomic_store(given_up, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        const float alpha = (float)block_sum(yv, redd[0]);
        if (done) break;
        double ww = 0.0;
#pragma unroll
        for (int q = 0; q < OWN; ++q) {
            y[q] = y[q] - alpha * v[q] - beta_p * vp[q];
            ww += (double)y[q] * (double)y[q];
        }
        const float beta = (float)sqrt(block_sum(ww, redd[1]));
        if (!(beta < 3.0e38f) || !(fabsf(alpha) < 3.0e38f)) {         // non-finite input, or a wait that was given up (uniform)
            settled = gave_up == 0;
            rho = NAN;
            break;
        }
        const float inv = beta > 0.0f ? 1.0f / beta : 0.0f;
#pragma unroll
        for (int q = 0; q < OWN; ++q) {
            const int i = tid + LC_THREADS * q;
            vp[q] = v[q];
            v[q] = y[q] * inv;
            if (i < 256 * NI) v_lds[i] = v[q];
        }
        beta_p = beta;
        if (tid == 0) { la[j] = alpha; lb[j] = beta; }
        __syncthreads();
        // the recurrence is looked at by one wavefront while the others go on to the next product: they stop one step later
        // than they could
        if (wave == 0) stop = lanczos_advance(rho, small, la, lb, j, beta, tol2);
    }
    if (member == 0 && tid == 0) { S.rho = rho; S.pm_done = settled ? 1 : 0; }
}

__global__ __launch_bounds__(LC_THREADS, 3) void lanczos_cluster_kernel(const FactorDev *fd, FactorScal *fs, const uint2 *map, int *ticket, float tol2, int steps,
                                                                        LanczosWaits waits)
{
    __shared__ int mine;
    if (threadIdx.x == 0) {
        const int t = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        mine = __hip_atomic_load(ticket + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ? -1 : t;
    }
    __syncthreads();
    if (mine < 0) return;
    const uint2 m = map[__builtin_amdgcn_readfirstlane(mine)];
    const FactorDev &F = fd[m.x];
    FactorScal &S = fs[m.x];
    if (F.n <= 512) lanczos_member<2>(F, S, (int)m.y, tol2, steps, waits, ticket + 1);
    else if (F.n <= 1024) lanczos_member<4>(F, S, (int)m.y, tol2, steps, waits, ticket + 1);
    else lanczos_member<8>(F, S, (int)m.y, tol2, steps, waits, ticket + 1);
}

// All steps of a factor of at most LC_MAX_N rows by one workgroup of 256 threads, dense or packed, from memory: for what
// lanczos_cluster_kernel left.  Rare, so short rather than fast; the vectors lie where the exchange did.
__device__ inline void lanczos_alone(const FactorDev &F, FactorScal &S, float tol2, int steps)
{
    __shared__ double red[4];
    __shared__ __align__(16) float la[LZ_MAX], lb[LZ_MAX];
    __shared__ int done;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = F.n;
    float *v = reinterpret_cast<float *>(F.lz_words), *vp = v + n, *y = vp + n;
    auto block_sum = [&](double x) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
        __syncthreads();
        if (lane == 0) red[wave] = x;
        __syncthreads();
        return red[0] + red[1] + red[2] + red[3];
    };
    double s = 0.0;
    for (int i = tid; i < n; i += 256) {
        v[i] = hash_unit(0u, (uint32_t)i); vp[i] = 0.0f;
        s += (double)v[i] * (double)v[i];
    }
    s = block_sum(s);
    const float inv0 = s > 0.0 ? (float)(1.0 / sqrt(s)) : 0.0f;
    for (int i = tid; i < n; i += 256) v[i] *= inv0;
    if (tid == 0) { done = 0; S.rho = 0.0f; S.lz_small = 0; }
    __syncthreads();
    float beta_p = 0.0f;
    for (int j = 0; j < steps; ++j) {
        double saa = 0.0, str = 0.0;
        for (int r = wave; r < n; r += 4) {
            float t = 0.0f;
            for (int c = lane; c < n; c += 64) {
                const float a = F.A[F.a_packed ? (c / PACK_T <= r / PACK_T ? packed_off(r, c) : packed_off(c, r)) : (size_t)r * F.lda + c];
                t += a * v[c];
                saa += (double)a * (double)a;
                if (c == r) str += (double)a;
            }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
            if (lane == 0) y[r] = t;
        }
        if (j == 0) {
            saa = block_sum(saa);
            str = block_sum(str);
            if (tid == 0) { S.fro2 = saa; S.trace = str; }
        }
        __syncthreads();
        double yv = 0.0, ww = 0.0;
        for (int i = tid; i < n; i += 256) yv += (double)(y[i] * v[i]);
        const float alpha = (float)block_sum(yv);
        for (int i = tid; i < n; i += 256) {
            y[i] = y[i] - alpha * v[i] - beta_p * vp[i];
            ww += (double)y[i] * (double)y[i];
        }
        const float beta = (float)sqrt(block_sum(ww));
        if (!(beta < 3.0e38f) || !(fabsf(alpha) < 3.0e38f)) {         // non-finite input (uniform)
            if (tid == 0) S.rho = NAN;
            break;
        }
        const float inv = beta > 0.0f ? 1.0f / beta : 0.0f;
        for (int i = tid; i < n; i += 256) { vp[i] = v[i]; v[i] = y[i] * inv; }
        beta_p = beta;
        if (tid == 0) { la[j] = alpha; lb[j] = beta; }
        __syncthreads();
        if (wave == 0 && lanczos_advance(S, la, lb, j, beta, tol2) && lane == 0) done = 1;
        __syncthreads();
        if (done) break;
    }
}

// ---- one launch per step -------------------------------------------------------------------------------
// Grid: x = row block, plus one that keeps the recurrence; y = factor.  Launch j: v_j from step j - 1, y_j = A v_j.
__global__ __launch_bounds__(256) void lanczos_step_kernel(const FactorDev *fd, FactorScal *fs, float tol2, int j, int blocks)
{
    const int f = blockIdx.y;
    FactorScal &S = fs[f];
    if (j > 0 && S.pm_done) return;
    const FactorDev &F = fd[f];
    const bool keeper = (int)blockIdx.x == blocks;
    if (!keeper && (int)blockIdx.x >= F.pm_blocks) return;
    const int n = F.n, lda = F.ldw;
    extern __shared__ __align__(16) float lz_smem[];
    float *v = lz_smem;
    __shared__ double redd[4];
    __shared__ float red[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    auto block_sum = [&](double x) -> double {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
        __syncthreads();
        if (lane == 0) redd[wave] = x;
        __syncthreads();
        return redd[0] + redd[1] + redd[2] + redd[3];
    };
    float alpha = 0.0f, beta = 0.0f;
    double ww = 0.0;
    if (j == 0) {
        for (int i = tid; i < n; i += 256) { const float x = hash_unit(0u, (uint32_t)i); v[i] = x; ww += (double)x * (double)x; }
    } else {
        double yv = 0.0;
        for (int b = tid; b < F.pm_blocks; b += 256) yv += (double)F.pm_partial[((j - 1) & 1) * F.pm_blocks + b];
        alpha = (float)block_sum(yv);
        const float *__restrict__ y = F.py[(j - 1) & 1], *__restrict__ v1 = F.pv[(j - 1) % 3], *__restrict__ v2 = F.pv[(j + 1) % 3];
        const float beta_p = j > 1 ? S.lz_b[j - 2] : 0.0f;
        for (int i = tid; i < n; i += 256) {
            float x = y[i] - alpha * v1[i];
            if (j > 1) x -= beta_p * v2[i];
            v[i] = x;
            ww += (double)x * (double)x;
        }
    }
    ww = block_sum(ww);
    beta = (float)sqrt(ww);
    const float inv = beta > 0.0f ? 1.0f / beta : 0.0f;
    for (int i = tid; i < n; i += 256) v[i] *= inv;
    __syncthreads();
    if (keeper) {
        for (int i = tid; i < n; i += 256) F.pv[j % 3][i] = v[i];
        if (j == 0) {
            if (tid == 0) { S.rho = 0.0f; S.lz_small = 0; S.pm_done = 0; }
            return;
        }
        if (j == 1) {
            double aa = 0.0, tr = 0.0;
            for (int b = tid; b < F.pm_blocks; b += 256) { const double2 q = F.pm_partial2[b]; aa += q.x; tr += q.y; }
            aa = block_sum(aa);
            tr = block_sum(tr);
            if (tid == 0) { S.fro2 = aa; S.trace = tr; }
        }
        if (!(beta < 3.0e38f) || !(fabsf(alpha) < 3.0e38f)) {
            if (tid == 0) { S.rho = NAN; S.pm_done = 1; }
            return;
        }
        __shared__ __align__(16) float la[LZ_MAX], lb[LZ_MAX];
        if (tid < j - 1) { la[tid] = S.lz_a[tid]; lb[tid] = S.lz_b[tid]; }
        if (tid == 0) { S.lz_a[j - 1] = la[j - 1] = alpha; S.lz_b[j - 1] = lb[j - 1] = beta; }
        __syncthreads();
        if (wave == 0) {
            const bool stop = lanczos_advance(S, la, lb, j - 1, beta, tol2);
            if (lane == 0 && stop) S.pm_done = 1;
        }
        return;
    }
    const float *__restrict__ A = F.Aw;
    const bool vec = ((reinterpret_cast<uintptr_t>(A) & 15u) == 0) && ((lda & 3) == 0);
    float syv = 0.0f;
    double saa = 0.0, str = 0.0;                             // every lane its part of the squares, lane 0 the diagonal
    const int base = blockIdx.x * LZ_ROWS + wave * (LZ_ROWS / 4);
#pragma unroll 1
    for (int rr = 0; rr < LZ_ROWS / 4; rr += 4) {
        const int r0 = base + rr;
        if (r0 >= n) break;
        float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        const float *a0 = A + (size_t)r0 * lda, *a1 = A + (size_t)min(r0 + 1, n - 1) * lda;
        const float *a2 = A + (size_t)min(r0 + 2, n - 1) * lda, *a3 = A + (size_t)min(r0 + 3, n - 1) * lda;
        const double m1 = r0 + 1 < n ? 1.0 : 0.0, m2 = r0 + 2 < n ? 1.0 : 0.0, m3 = r0 + 3 < n ? 1.0 : 0.0;
        int c0 = 0;
        if (vec) {
            const int n4 = n >> 2;
#pragma unroll 2
            for (int c = lane; c < n4; c += 64) {
                const float4 x = reinterpret_cast<const float4 *>(v)[c];
                const float4 t0 = reinterpret_cast<const float4 *>(a0)[c], t1 = reinterpret_cast<const float4 *>(a1)[c];
                const float4 t2 = reinterpret_cast<const float4 *>(a2)[c], t3 = reinterpret_cast<const float4 *>(a3)[c];
                s[0] += t0.x * x.x + t0.y * x.y + t0.z * x.z + t0.w * x.w;
                s[1] += t1.x * x.x + t1.y * x.y + t1.z * x.z + t1.w * x.w;
                s[2] += t2.x * x.x + t2.y * x.y + t2.z * x.z + t2.w * x.w;
                s[3] += t3.x * x.x + t3.y * x.y + t3.z * x.z + t3.w * x.w;
                if (j == 0) saa += square_sum(t0) + m1 * square_sum(t1) + m2 * square_sum(t2) + m3 * square_sum(t3);
            }
            c0 = n4 << 2;
        }
#pragma unroll 4
        for (int c = c0 + lane; c < n; c += 64) {
            const float x = v[c];
            s[0] += a0[c] * x; s[1] += a1[c] * x; s[2] += a2[c] * x; s[3] += a3[c] * x;
            if (j == 0) {
                const double t0 = (double)a0[c], t1 = (double)a1[c], t2 = (double)a2[c], t3 = (double)a3[c];
                saa += t0 * t0 + m1 * t1 * t1 + m2 * t2 * t2 + m3 * t3 * t3;
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) s[e] += __shfl_xor(s[e], off, 64);
            if (r0 + e < n) {
                syv += s[e] * v[r0 + e];
                if (lane == 0) F.py[j & 1][r0 + e] = s[e];
                if (j == 0) str += (double)A[(size_t)(r0 + e) * lda + r0 + e];
            }
        }
    }
    if (lane == 0) red[wave] = syv;
    __syncthreads();
    if (tid == 0) F.pm_partial[(j & 1) * F.pm_blocks + blockIdx.x] = red[0] + red[1] + red[2] + red[3];
    if (j == 0) {
        saa = block_sum(saa);
        str = block_sum(lane == 0 ? str : 0.0);
        if (tid == 0) F.pm_partial2[blockIdx.x] = make_double2(saa, str);
    }
}

// Full copy of packed statistics for the workgroup-per-factor kernel: 128 x 128 stored tiles, their mirror images
// through LDS.  Grid: x = lower tile, y = factor.
__global__ __launch_bounds__(256) void lanczos_unpack_kernel(const FactorDev *fd)
{
    const FactorDev &F = fd[blockIdx.y];
    if (!F.a_packed || (int)blockIdx.x >= F.ntri) return;
    int ti, tj;
    tri_decode((int)blockIdx.x, ti, tj);
    const float *tile = F.A + (size_t)blockIdx.x * PACK_T * PACK_T;
    float *dst = const_cast<float *>(F.Aw);
    const int n = F.n, ld = F.ldw, tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    __shared__ float s[32][33];
    for (int sub = 0; sub < 16; ++sub) {
        const int r0 = (sub >> 2) * 32, c0 = (sub & 3) * 32;
        __syncthreads();
        for (int r = ty; r < 32; r += 8) {
            const float x = tile[(r0 + r) * PACK_T + c0 + tx];
            s[r][tx] = x;
            const int gr = ti * PACK_T + r0 + r, gc = tj * PACK_T + c0 + tx;
            if (gr < n && gc < n) dst[(size_t)gr * ld + gc] = x;
        }
        __syncthreads();
        if (ti != tj)
            for (int r = ty; r < 32; r += 8) {
                const int gr = tj * PACK_T + c0 + r, gc = ti * PACK_T + r0 + tx;
                if (gr < n && gc < n) dst[(size_t)gr * ld + gc] = s[tx][r];
            }
    }
}

}  // namespace asteria
