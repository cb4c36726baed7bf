// Per-factor device state of asteria_inverse_root, shared by its kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace asteria {

constexpr int LZ_MAX = 128;   // most Lanczos steps of the lambda_max estimate (size of the recurrence kept per factor)

enum : int { ST_RUN = 0, ST_LAST = 1, ST_DONE = 2, ST_FAIL = 3 };
// what the chain products of a factor run on in the current iteration
enum : int { TIER_F64 = 0, TIER_DIGIT = 1, TIER_PAIR = 2 };

// Workgroups of lanczos_cluster_kernel ("members") that share a factor.
constexpr int LC_WAVES = 12, LC_THREADS = 64 * LC_WAVES, LC_MAX_N = 2048;
__host__ __device__ inline int lanczos_rows(int n) { return LC_WAVES * (n <= 512 ? 16 : (n <= 1024 ? 8 : 4)); }     // of a member
__host__ __device__ inline int lanczos_members(int n) { return (n + lanczos_rows(n) - 1) / lanczos_rows(n); }
// Whether the largest factor's members find room on `cus` compute units (a member fills one) beside those of three other calls, on other
// streams or of other processes: only what waits at the frontier of each call counts.  A whole MI355X has room for 43; 32 CUs
// of it for the 8 of n = 768.
__host__ __device__ inline bool lanczos_cluster_room(int n_max, int cus) { return n_max <= LC_MAX_N && 4 * lanczos_members(n_max) <= cus; }
// words of a factor's exchange: two buffers of n, and each member's partial sums of squares and of the diagonal as halves of doubles
__host__ __device__ inline size_t lanczos_words(int n) { return 2 * (size_t)n + 4 * (size_t)lanczos_members(n); }

struct FactorDev {
    const float *A;
    float *Xout;
    // plane path
    char *X[2];         // pair planes: X_k in X[k & 1]
    char *P[4];         // pair planes of the chain, slots as in root_products.h
    char *D[4];         // digit planes of the chain, the same slots
    double *F[4];       // fp64 matrices of the chain, the same slots
    int *flags;         // [0]: an entry left the range of its digits
    int rowb;           // bytes of a pair plane row
    int npart;          // entries of `partial` and `qpart`
    float *qpart;       // per tile: sum q(M)^2 of the test before the last update
    int tile_start_p;   // first tile of this factor in the launches of the pair products
    // fp32 / fp64 path
    float *X32b;        // second fp32 X buffer (workspace); X is kept in fp32 in every precision tier
    float *M32[2];
    float *T32;
    float *T432;
    double *M64[2];
    double *T64;
    union {
        double *T464;
        uint64_t *lz_words;   // plane path: exchange of lanczos_cluster_kernel
    };
    // both
    const float *Aw;    // A in full storage as the lambda_max estimate reads it: A, or a copy of packed statistics
    int ldw;
    float *pv[3];       // Lanczos vectors (packed statistics: the current one, the one before it, A times the current one)
    float *py[2];       // A times the vectors of the last two steps
    float *pm_partial;  // per mat-vec workgroup: sum y v; two steps' in turn
    double2 *pm_partial2; // per mat-vec workgroup, first step only: (sum a_ij^2, sum a_ii)
    float *partial;     // per lower-triangle tile: sum (M - I)^2 (2 ntri entries: a second one per tile for kernels that split tiles)
    int n, lda, ldx;
    union {
        int ld32;           // fp32 / fp64 path
        int lz_start;       // plane path: first of this factor's workgroups in lanczos_cluster_kernel
    };
    int ld64;
    int ntri;           // lower-triangle tiles
    int tile_start;     // first tile of this factor in tile-indexed launches
    int pm_blocks;
    float eps_in;
    int a_packed;       // A lies in packed lower tiles (gemm.h, packed_off): lda unused
    float *pm_tile;     // packed A: per lower tile 2 x 128 partial products of the mat-vec and the sum of a^2 as a double
};

// coefficients of one product of the plane path: C = own1 O1 + own2 O2 + gam A B, in values
struct RootProd { double own1, own2, gam; };

struct FactorScal {
    float lam;       // lambda_max estimate
    float eps;       // absolute eps used
    float scale;     // s
    float resid;     // last ||M - I||_F
    float rho;       // largest Ritz value so far: the lambda_max estimate
    int lz_small;    // consecutive steps that moved the estimate by less than the tolerance
    int iters;       // X updates performed / scheduled
    int xloc;        // 0: current fp32 X in Xout, 1: in X32b (plane path: only its lower triangle in Xout)
    int info;
    int pm_done;
    float lo, hi;    // interval assumed to contain the spectrum of the current M
    float ca, cg;    // coefficients of the current T = ca I - cg M
    float coef_next[2];   // coefficients the M-update epilogue uses for the next T
    // ||A||_F^2 and tr(A), gathered during the first mat-vec of the lambda_max estimate; squares of fp32 numbers do
    // not fit fp32 for statistics of the size of 1e-20
    double fro2, trace;
    float x_scale;        // power of two that brings X into the fp16 range for the 16-bit products
    // (lo, hi) of the M the current iteration starts from and the g of its T: lo, hi, ca, cg above
    // are advanced to the next iteration's before the products of the current one run
    float lo_cur, hi_cur, cg_cur;
    float lz_a[LZ_MAX], lz_b[LZ_MAX];   // the Lanczos recurrence: diagonal and off-diagonal of the tridiagonal matrix
    // plane path
    int tier, next_tier;
    int ns, levels;       // digits of this factor's digit planes (4 or 5), digit-product levels kept in this iteration
    int from_f64;         // this iteration's digits of M are made from the fp64 one
    int swapped;          // ... and lie in slot 1 since, E2's in slot 0
    int handover;         // the M-update of this iteration writes pair planes for the next one
    int pair_m;           // ... and pair planes beside the digits (the next T is linear: X' = a X - b X M)
    int dexp[5];          // exponents of the digit planes' quanta by slot; 4: the next M
    double lo_d, hi_d;    // interval of the current M
    double dmax;          // bound on the largest diagonal entry of M
    float x1a, x1s, x1b;  // X_1 = x1a I - x1s E (times x_scale); E = x1b M where T is linear
    RootProd prod[7];     // by RootOp
    // test before the last update (plane_advance): q = q[0] I + q[1] M + q[2] M^2 + q[3] E, bound on its squares; 0: none
    float q[4], q_limit;
};

// Sum of `count` numbers by one wavefront, the same bits from every one.
__device__ __forceinline__ float wave_total(const float *p, int count)
{
    float t = 0.0f;
    for (int i = threadIdx.x & 63; i < count; i += 64) t += p[i];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
    return t;
}

// State of a factor once the last iteration's E is there: the iteration goes on where the test does not hold.
__device__ __forceinline__ int state_after_test(const FactorDev &F, const FactorScal &S, int st)
{
    return st == ST_LAST && S.q_limit > 0.0f && !(wave_total(F.qpart, F.npart) <= S.q_limit) ? ST_RUN : st;
}

}  // namespace asteria
