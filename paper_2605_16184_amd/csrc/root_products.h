// The products of the coupled root iteration on plane storage (planes.h): one kernel on pair planes (fp16
// matrix cores), one on digit planes (int8 matrix cores).  Every product is symmetric and has the form
//     C = k1 O1 + k2 O2 + g A B        (A, B, O1, O2, C symmetric, commuting)
// with per-factor coefficients that the control kernel has left on the device; only tiles on or below the
// diagonal are computed, their mirror images are stored with them.
#pragma once
#include "planes.h"
#include "root_factor.h"

namespace asteria {

typedef int i32x16 __attribute__((ext_vector_type(16)));

// Which product a launch computes.  M lies in slot 0, M^2 and then T^2's complement in slot 1, E in slot 2, T^2 M in
// slot 3; the next M takes the slot of M.
//
// T^4 M is formed as T^2 (T^2 M): the same number of products as with T^4, and what the storage of its operands loses
// is of the size of T^2 <= a^2 times the large eigenvalues of T^2 M (about 1) instead of T^4 <= a^4 = 113 times those of
// M, against the small eigenvalues that the map lifts.  Error of the root against 64 bits that does not commute with A
// (per eigen-direction, n = 1024, eps = 1e-8), with T^4 and so: rows scaled over 4 decades 1.2e-4 and 1.0e-5, power law
// 1.2e-5 and 4.3e-6.
enum RootOp : int {
    OP_SQ = 0,   // E  = b M - c M M                      (T of degree 2)
    OP_SQ3,      // M2 = M M                              (T of degree 3, first product)
    OP_CUBE,     // E  = b M - c M2 + d M2 M              (... second product)
    OP_E2,       // E2 = 2 a E - E E,    T^2 = a^2 I - E2
    OP_W,        // W  = a^2 M - E2 M = T^2 M
    OP_M,        // M' = a^2 W - E2 W
    OP_X,        // X' = a X - X E
    OP_COUNT
};

// fp16 scales of the pair planes.  The spectra are bounded by M: 2.02, M^2: 4.1, E: a, E2: a^2, W = (M' M)^(1/2): 2.02
// with a <= 3.6 for every coefficient set in use, and |entry| <= largest diagonal entry <= ||.||_2.
constexpr float PAIR_SCALE_M = 8192.0f, PAIR_SCALE_M2 = 8192.0f, PAIR_SCALE_E = 8192.0f, PAIR_SCALE_E2 = 2048.0f, PAIR_SCALE_W = 8192.0f;

struct RootOperands {
    int A, B, O1, O2, C;     // slots (O2 = -1: none)
};
__device__ __forceinline__ RootOperands root_operands(int op, bool linear)
{
    const int e = linear ? 0 : 2;        // T of degree 1: E is b M and takes M's place in the products
    switch (op) {
    case OP_SQ: return {0, 0, 0, -1, 2};
    case OP_SQ3: return {0, 0, -1, -1, 1};
    case OP_CUBE: return {1, 0, 0, 1, 2};
    case OP_E2: return {e, e, e, -1, 1};
    case OP_W: return {1, 0, 0, -1, 3};
    default: return {1, 3, 3, -1, 0};              // OP_M
    }
}
__device__ __forceinline__ float pair_scale_of(int op, int slot)
{
    switch (slot) {
    case 0: return PAIR_SCALE_M;
    case 1: return (op == OP_SQ3 || op == OP_CUBE) ? PAIR_SCALE_M2 : PAIR_SCALE_E2;
    case 2: return PAIR_SCALE_E;
    default: return PAIR_SCALE_W;
    }
}

// XCD-aware order: workgroup b lands on XCD b % 8; every XCD takes a contiguous range of tiles, so the tiles of
// one factor share an L2
__device__ __forceinline__ int xcd_tile(int total)
{
    const int per = (total + NUM_XCD - 1) / NUM_XCD;
    return (int)(blockIdx.x % NUM_XCD) * per + (int)(blockIdx.x / NUM_XCD);
}

__device__ __forceinline__ void store_partial(float rsum, float *red, float *dst, int lane, int wave, int tid, int waves)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) rsum += __shfl_xor(rsum, off, 64);
    if (lane == 0) red[wave] = rsum;
    __syncthreads();
    if (tid == 0) {
        float t = 0.0f;
        for (int w = 0; w < waves; ++w) t += red[w];
        *dst = t;
    }
}

// ---- pair planes -------------------------------------------------------------------------------------
// A workgroup of 2 x 2 wavefronts, WT x WT MFMA blocks each (tile 64 WT), slabs of 32 k: three fp16 MFMA passes
// per block and 16 k (lo hi, hi lo, hi hi: both operands to 2^-22), fp32 sums.  Operands go from memory to LDS
// without passing through registers; ST stages.
//   WT = 2, two stages: 64 KiB of LDS, two workgroups per CU, one loading or storing while the other multiplies.
//     600 symmetric products of n = 1024: K loop 2.0 ms (1.0 PFLOP/s issued; the fp16 library product of
//     8192^3 reaches 1.07 on the same card), against 2.6 ms when the fp32 operands are split in the loop (both with one
//     sum for all terms; whole launches of the refresh of the 1.1B model, as they are now: 0.71 PFLOP/s issued).
//     256 x 256 tiles on 8 wavefronts: the same within 2 % at n = 1024 and 4 % slower at n = 512.
//   WT = 1, four stages: for launches of too few 128-wide tiles to fill the chip; short K steps, so the loads
//     need more than one slab of lead.
// In a diagonal tile the wavefront above the diagonal multiplies nothing, the two on it three of four blocks.
template <int WT, int ST>
__global__ __launch_bounds__(256, 2) void pair_product_kernel(const FactorDev *__restrict__ fd, const FactorScal *__restrict__ fs,
                                                              const int *__restrict__ state, const uint2 *__restrict__ map, int total,
                                                              int op0, int op1, int k, int degree)
{
    constexpr int T = 64 * WT;
    using Loader = PlaneLoader<8, T, T, 4>;
    extern __shared__ __align__(16) unsigned char plane_smem[];
    ASTERIA_LDS char *lds = (ASTERIA_LDS char *)plane_smem;
    const int all = op1 >= 0 ? 2 * total : total;
    const int w = xcd_tile(all);
    if (w >= all) return;
    // the two products of a double launch alternate tile by tile: they share the rows of E
    const int op = (op1 >= 0 && (w & 1)) ? op1 : op0;
    const uint2 tile = map[op1 >= 0 ? w >> 1 : w];
    const int f = (int)tile.x;
    const FactorScal &S = fs[f];
    if (op != OP_X && S.tier != TIER_PAIR) return;
    const FactorDev &F = fd[f];
    const bool makes_e = op == OP_SQ || op == OP_SQ3 || op == OP_CUBE;
    const int st = makes_e ? state[f] : state_after_test(F, S, state[f]);
    if (st != ST_RUN && !(st == ST_LAST && (makes_e || op == OP_X))) return;
    const int ti = (int)(tile.y >> 16), tj = (int)(tile.y & 0xffffu);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1, r = lane & 31, h = lane >> 5;
    const int n = F.n, rowb = F.rowb, p = k & 1, row0 = ti * T, col0 = tj * T;
    const char *A, *B, *O1 = nullptr, *O2 = nullptr;
    char *C;
    float sA, sB, s1 = 1.0f, s2 = 1.0f, sC;
    if (op == OP_X) {
        A = F.X[p]; B = F.P[degree == 1 ? 0 : 2]; C = F.X[p ^ 1];
        sA = sC = S.x_scale; sB = degree == 1 ? PAIR_SCALE_M : PAIR_SCALE_E;
    } else {
        const RootOperands o = root_operands(op, degree == 1);
        A = F.P[o.A]; B = F.P[o.B]; C = F.P[o.C];
        sA = pair_scale_of(op, o.A); sB = pair_scale_of(op, o.B);
        if (o.O1 >= 0) { O1 = F.P[o.O1]; s1 = pair_scale_of(op, o.O1); }
        if (o.O2 >= 0) { O2 = F.P[o.O2]; s2 = pair_scale_of(op, o.O2); }
        sC = pair_scale_of(op, o.C);
    }
    const RootProd pc = S.prod[op];
    const float k1 = (float)(pc.own1 * (double)(sC / s1)), k2 = (float)(pc.own2 * (double)(sC / s2));
    const float kg = (float)(pc.gam * (double)sC / ((double)sA * (double)sB));

    // the cross terms, 2^-11 of the leading ones, in sums of their own: a third of the roundings at full size (log-spaced
    // spectrum, n = 1024, eps = 1e-6: error as above 5.2e-4 with one sum, 3.3e-4 with two; the time of a refresh + 1 %)
    floatx16 acc[WT][WT], cross[WT][WT];
#pragma unroll
    for (int i = 0; i < WT; ++i)
#pragma unroll
        for (int j = 0; j < WT; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = cross[i][j][v] = 0.0f;

    Loader ld;
    ld.init(A, B, rowb, n, row0, col0, wave, lane);
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
    const int nk = plane_groups(n), last = nk - 1;
    const int sw = plane_swz<8>(r);
    const ASTERIA_LDS char *fa = lds + (wm * WT * 32 + r) * 128, *fb = lds + (T + wn * WT * 32 + r) * 128;
    const int diag_d = ti == tj ? wm - wn : 1;        // < 0: above the diagonal, 0: on it
    auto mma = [](u32x4 a, u32x4 b, floatx16 c) __attribute__((always_inline)) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(pl_f16x8, a), __builtin_bit_cast(pl_f16x8, b), c, 0, 0, 0);
    };
    auto compute = [&](uint32_t stage) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            u32x4 ah[WT], al[WT], bh[WT], bl[WT];
            const int ch = ((s * 2 + h) ^ sw) * 16, cl = ((4 + s * 2 + h) ^ sw) * 16;
#pragma unroll
            for (int j = 0; j < WT; ++j) {
                bh[j] = *(const ASTERIA_LDS u32x4 *)(fb + stage + j * 4096 + ch);
                bl[j] = *(const ASTERIA_LDS u32x4 *)(fb + stage + j * 4096 + cl);
            }
#pragma unroll
            for (int i = 0; i < WT; ++i) {
                ah[i] = *(const ASTERIA_LDS u32x4 *)(fa + stage + i * 4096 + ch);
                al[i] = *(const ASTERIA_LDS u32x4 *)(fa + stage + i * 4096 + cl);
            }
#pragma unroll
            for (int i = 0; i < WT; ++i) {
                const bool cut = WT == 2 && i == 0 && diag_d == 0;      // block (0, 1) of a wavefront on the diagonal
#pragma unroll
                for (int j = 0; j < WT; ++j) if (!(j == 1 && cut)) cross[i][j] = mma(al[i], bh[j], cross[i][j]);
#pragma unroll
                for (int j = 0; j < WT; ++j) if (!(j == 1 && cut)) cross[i][j] = mma(ah[i], bl[j], cross[i][j]);
#pragma unroll
                for (int j = 0; j < WT; ++j) if (!(j == 1 && cut)) acc[i][j] = mma(ah[i], bh[j], acc[i][j]);
            }
        }
    };
    // The loads past the end repeat the last slab, so the number in flight is the same in every iteration.
#pragma unroll
    for (int q = 0; q < ST - 1; ++q) ld.issue(lds0 + q * Loader::STAGE, min(q, last));
    uint32_t cur = 0, nxt = (ST - 1) * Loader::STAGE;
    for (int kt = 0; kt < nk; ++kt) {
        wait_lds_loads<Loader::NI *(ST - 2)>();
        __builtin_amdgcn_s_barrier();                 // the slab has landed, and everyone is done with the one before
        ld.issue(lds0 + nxt, min(kt + ST - 1, last));
        if (diag_d >= 0) compute(cur);
        cur = cur + Loader::STAGE == ST * Loader::STAGE ? 0u : cur + Loader::STAGE;
        nxt = nxt + Loader::STAGE == ST * Loader::STAGE ? 0u : nxt + Loader::STAGE;
    }
    wait_lds_loads<0>();
    __builtin_amdgcn_s_barrier();                     // LDS is free for the stores

    ASTERIA_LDS uint32_t *ws = (ASTERIA_LDS uint32_t *)(lds + wave * PLANE_SCRATCH_BYTES);
    const bool to_user = op == OP_X && st == ST_LAST;
    const bool first_x = k == 0 && (op == OP_SQ || op == OP_CUBE);    // X_1 = X_0 T_0, X_0 a multiple of I
    const float inv_c = 1.0f / sC;
    const float x1a = S.x1a, x1e = -S.x1s * inv_c, inv_x = 1.0f / S.x_scale;
    ASTERIA_GLOBAL float *X = (ASTERIA_GLOBAL float *)F.Xout;
    const int ldx = F.ldx;
    // the test before the last update, by the product that completes E
    const bool test = st == ST_LAST && S.q_limit > 0.0f && ((op == OP_SQ && degree == 2) || op == OP_CUBE);
    const float q1 = S.q[1] / s1, q2 = S.q[2] / s2, q3 = S.q[3] * inv_c, q0 = S.q[0];
    float rsum = 0.0f;
    // X row-major: a block's base is uniform, beside a 32-bit offset of the lane
    const uint32_t xo = (uint32_t)(4 * h) * (uint32_t)ldx + (uint32_t)r;
#pragma unroll
    for (int i = 0; i < WT; ++i) {
#pragma unroll
        for (int j = 0; j < WT; ++j) {
            const int br = row0 + (wm * WT + i) * 32, bc = col0 + (wn * WT + j) * 32;
            if (br < bc || br >= n || bc >= n) continue;
            const bool diag = br == bc;
            acc[i][j] += cross[i][j];
            float val[16], q[16];
            if (O1) {
                load_pair_block(O1, rowb, n, br, bc, lane, val);
                if (test) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) q[v] = q1 * val[v];
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) val[v] = k1 * val[v] + kg * acc[i][j][v];
            } else if (op == OP_X) {
                if (!diag && br + 32 <= n) {
                    const ASTERIA_GLOBAL float *x = X + (size_t)br * ldx + bc;
#pragma unroll
                    for (int v = 0; v < 16; ++v) val[v] = (x + (size_t)(8 * (v >> 2) + (v & 3)) * ldx)[xo];
                } else {
                    const int col = bc + r;
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int row = br + 8 * (v >> 2) + 4 * h + (v & 3);
                        val[v] = row < n && col < n && row >= col ? X[(size_t)row * ldx + col] : 0.0f;
                    }
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) val[v] = k1 * val[v] + kg * acc[i][j][v];
            } else {
#pragma unroll
                for (int v = 0; v < 16; ++v) val[v] = kg * acc[i][j][v];
            }
            if (O2) {
                float o[16];
                load_pair_block(O2, rowb, n, br, bc, lane, o);
#pragma unroll
                for (int v = 0; v < 16; ++v) val[v] += k2 * o[v];
                if (test) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) q[v] += q2 * o[v];
                }
            }
            const int col = bc + r;
            if (op == OP_M) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = br + 8 * (v >> 2) + 4 * h + (v & 3);
                    const float er = val[v] * inv_c - (row == col ? 1.0f : 0.0f);
                    if (row < n && col < n && row >= col) rsum += row == col ? er * er : 2.0f * er * er;
                }
            }
            if (test) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = br + 8 * (v >> 2) + 4 * h + (v & 3);
                    const float x = q[v] + q3 * val[v] + (row == col ? q0 : 0.0f);
                    if (row < n && col < n && row >= col) rsum += row == col ? x * x : 2.0f * x * x;
                }
            }
            if (op == OP_X) {
                // X in fp32: its lower triangle until the last update, which completes the caller's matrix
                const bool vec = (ldx & 3) == 0 && (reinterpret_cast<uintptr_t>(F.Xout) & 15u) == 0;
                if (!diag && br + 32 <= n) {
                    ASTERIA_GLOBAL float *x = X + (size_t)br * ldx + bc;
#pragma unroll
                    for (int v = 0; v < 16; ++v) (x + (size_t)(8 * (v >> 2) + (v & 3)) * ldx)[xo] = val[v] * inv_c;
                } else {
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int row = br + 8 * (v >> 2) + 4 * h + (v & 3);
                        if (row < n && col < n && row >= col) X[(size_t)row * ldx + col] = val[v] * inv_c;
                    }
                }
                if (to_user && col < n) {
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const int rb = br + 8 * g + 4 * h;
                        floatx4 t;
#pragma unroll
                        for (int e = 0; e < 4; ++e) t[e] = val[4 * g + e] * inv_c;
                        if (!diag && vec && rb + 4 <= n) *(ASTERIA_GLOBAL floatx4 *)(X + (size_t)col * ldx + rb) = t;
                        else
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                if (rb + e < n && (!diag || rb + e > col)) X[(size_t)col * ldx + rb + e] = t[e];
                    }
                }
                if (to_user) continue;
            }
            uint32_t wd[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = br + 8 * (v >> 2) + 4 * h + (v & 3);
                wd[v] = (row < n && col < n) ? pair_word(val[v]) : 0u;
            }
            store_pair_block(C, rowb, n, br, bc, wd, lane, ws);
            if (first_x) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = br + 8 * (v >> 2) + 4 * h + (v & 3);
                    const float x = x1e * val[v] + (row == col ? x1a : 0.0f);
                    wd[v] = (row < n && col < n) ? pair_word(x) : 0u;
                    if (row < n && col < n && row >= col) X[(size_t)row * ldx + col] = x * inv_x;
                }
                store_pair_block(F.X[1], rowb, n, br, bc, wd, lane, ws);
            }
        }
    }
    if (op == OP_M || test) {
        __syncthreads();
        store_partial(rsum, reinterpret_cast<float *>(plane_smem), (test ? F.qpart : F.partial) + ti * (ti + 1) / 2 + tj, lane, wave, tid, 4);
    }
}

template <int WT, int ST>
inline hipError_t launch_pair_product(const FactorDev *fd, const FactorScal *fs, const int *state, const uint2 *map, int total,
                                      int op0, int op1, int k, int degree, hipStream_t stream)
{
    if (total <= 0) return hipSuccess;
    constexpr size_t stage = ST * (size_t)PlaneLoader<8, 64 * WT, 64 * WT, 4>::STAGE, epi = 4 * (size_t)PLANE_SCRATCH_BYTES;
    constexpr size_t lds = stage > epi ? stage : epi;
    auto kern = pair_product_kernel<WT, ST>;
    static bool configured[MAX_DEVICES] = {};
    if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kern), lds, configured); e != hipSuccess) return e;
    const int all = op1 >= 0 ? 2 * total : total, per = (all + NUM_XCD - 1) / NUM_XCD;
    profile_begin(224, stream);
    hipLaunchKernelGGL(kern, dim3(per * NUM_XCD), dim3(256), lds, stream, fd, fs, state, map, total, op0, op1, k, degree);
    profile_end(stream);
    return hipGetLastError();
}

// ---- digit planes ------------------------------------------------------------------------------------
// C = k1 O1 + g A B in exact integer arithmetic up to the level cut: with A = qa sum_s a_s 256^(NS-1-s) and B
// alike, the digit products of levels s + t < L are summed in int32 (|sum| <= L K 2^14 < 2^31 for K <= 21845),
// one accumulator per level.  The result is assembled in fp64 and rounded to the quantum of C, whose exponent
// the control kernel has taken from a bound on C's diagonal (|entry| <= largest diagonal entry: every matrix
// here is positive semi-definite).  (NS, L) is the control kernel's choice per factor and iteration:
//   (4, 4) 10, (4, 5) 13, (5, 5) 15, (5, 6) 19 int8 MFMA passes.
//
// A workgroup of 2 x 2 wavefronts of 32 BI x 32 (BI 32 x 32 MFMA blocks, L level accumulators each) computes one
// 128 x 64 half of a tile in 2 / BI steps, slabs of 32 k, two LDS stages of 24 KiB (NS = 4): two workgroups per
// CU, so that one multiplies while the other assembles and stores.  BI = 2 where the accumulators leave room
// for it in 256 registers (a third less LDS traffic per MFMA).
template <int NS, int L, int BI>
__device__ __forceinline__ void digit_tile(const FactorDev &F, const FactorScal &S, int op, int k, int degree, int ti, int tj, int half,
                                           unsigned char *smem)
{
    constexpr int CPR = 2 * NS, ROWL = CPR * 16, RB = 64 * BI;
    using Loader = PlaneLoader<CPR, RB, 64, 4>;
    ASTERIA_LDS char *lds = (ASTERIA_LDS char *)smem;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1, r = lane & 31, h = lane >> 5;
    const int n = F.n, col0 = tj * 128 + half * 64;
    if (col0 >= n) return;                            // nothing to store; the half's partial sum was cleared when it was last read
    const int rowb = digit_row_bytes(n, NS);
    const RootOperands o = root_operands(op, degree == 1);
    auto digits_of = [&](int slot) { return F.D[slot < 2 ? slot ^ S.swapped : slot]; };
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
    const int nk = plane_groups(n), last = nk - 1;
    const int sw = plane_swz<CPR>(r);
    ASTERIA_LDS uint32_t *ws = (ASTERIA_LDS uint32_t *)(lds + wave * PLANE_SCRATCH_BYTES);
    const RootProd pc = S.prod[op];
    // value of an operand = integer * 2^dexp; lowest kept level of the product = 256^(2 (NS - 1) - (L - 1)) quanta
    const double qo = ldexp(1.0, S.dexp[o.O1]), qab = ldexp(1.0, S.dexp[o.A] + S.dexp[o.B] + 8 * (2 * NS - 1 - L));
    const double c1 = pc.own1 * qo, cg = pc.gam * qab;
    const double inv_q = ldexp(1.0, -S.dexp[op == OP_M ? 4 : o.C]);   // exponent slot 4: the next M
    const bool to_digits = !(op == OP_M && S.handover);
    // E feeds the X update as pair planes too (k > 0); so does M where T is linear or where the fp16 tier takes over
    const bool to_pair = (op == OP_SQ && k > 0) || (op == OP_M && (S.handover || S.pair_m));
    const bool first_x = op == OP_SQ && k == 0;       // X_1 = X_0 T_0, X_0 a multiple of I
    const double pe = first_x ? -(double)S.x1s : (op == OP_M ? (double)PAIR_SCALE_M : (double)PAIR_SCALE_E);
    const double pd = first_x ? (double)S.x1a : 0.0, inv_x = 1.0 / (double)S.x_scale;
    float rsum = 0.0f;
    bool over = false;
#pragma unroll 1
    for (int step = 0; step < 2 / BI; ++step) {
        const int row0 = ti * 128 + step * 64;
        if (row0 >= n || row0 + RB - 1 < col0) continue;              // nothing of it below the diagonal (uniform)
        Loader ld;
        ld.init(digits_of(o.A), digits_of(o.B), rowb, n, row0, col0, wave, lane);
        const ASTERIA_LDS char *fa = lds + (wm * 32 * BI + r) * ROWL, *fb = lds + (RB + wn * 32 + r) * ROWL;
        i32x16 acc[L][BI];
#pragma unroll
        for (int l = 0; l < L; ++l)
#pragma unroll
            for (int i = 0; i < BI; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[l][i][v] = 0;
        const bool above = row0 + (wm + 1) * 32 * BI - 1 < col0 + wn * 32;     // this wavefront's part lies above the diagonal
        auto compute = [&](uint32_t stage) {
            i32x4 a[NS][BI], b[NS];
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const int c = ((2 * s + h) ^ sw) * 16;
                b[s] = *(const ASTERIA_LDS i32x4 *)(fb + stage + c);
#pragma unroll
                for (int i = 0; i < BI; ++i) a[s][i] = *(const ASTERIA_LDS i32x4 *)(fa + stage + i * 32 * ROWL + c);
            }
            // consecutive MFMAs write different accumulators
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int t = 0; t < NS; ++t) {
                    if (s + t >= L) continue;
#pragma unroll
                    for (int i = 0; i < BI; ++i) acc[s + t][i] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[s][i], b[t], acc[s + t][i], 0, 0, 0);
                }
        };
        ld.issue(lds0, 0);
        uint32_t cur = 0;
        for (int kt = 0; kt < nk; ++kt) {
            wait_lds_loads<0>();
            __builtin_amdgcn_s_barrier();
            const uint32_t nxt = cur ? 0u : (uint32_t)Loader::STAGE;
            ld.issue(lds0 + nxt, min(kt + 1, last));
            if (!above) compute(cur);
            cur = nxt;
        }
        wait_lds_loads<0>();
        __builtin_amdgcn_s_barrier();
#pragma unroll
        for (int i = 0; i < BI; ++i) {
            const int br = row0 + (wm * BI + i) * 32, bc = col0 + wn * 32;
            if (br < bc || br >= n || bc >= n) continue;
            const int col = bc + r;
            const char *own = digits_of(o.O1) + (size_t)min(col, n - 1) * rowb + (br >> 5) * (32 * NS) + 4 * h;
            // calls use(v, row, value) for the block's elements; used once per output format (the second time
            // the own digits come from L1: cheaper than holding both formats in registers)
            auto values = [&](auto use) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    double ov[4];
                    load_digit_group<NS>(own, g, ov);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int v = 4 * g + e, row = br + 8 * g + 4 * h + e;
                        double t = (double)acc[0][i][v];
#pragma unroll
                        for (int l = 1; l < L; ++l) t = t * 256.0 + (double)acc[l][i][v];
                        const double val = c1 * ov[e] + cg * t;
                        use(v, row, (row < n && col < n) ? val : 0.0);
                    }
                }
            };
            if (to_digits) {
                uint32_t wd[16], tp[16];
                values([&](int v, int, double val) { wd[v] = digit_word<NS>(rint(val * inv_q), tp[v], over); });
                store_digit_block<NS>(digits_of(o.C), rowb, n, br, bc, wd, tp, lane, ws);
            }
            if (to_pair || first_x) {
                uint32_t pw[16];
                values([&](int v, int row, double val) {
                    const double x = pe * val + (row == col ? pd : 0.0);
                    pw[v] = (row < n && col < n) ? pair_word((float)x) : 0u;
                    if (first_x && row < n && col < n && row >= col) F.Xout[(size_t)row * F.ldx + col] = (float)(x * inv_x);
                });
                store_pair_block(first_x ? F.X[1] : F.P[o.C], F.rowb, n, br, bc, pw, lane, ws);
            }
            if (op == OP_M)
                values([&](int, int row, double val) {
                    const float er = (float)(val - (row == col ? 1.0 : 0.0));
                    if (row < n && col < n && row >= col) rsum += row == col ? er * er : 2.0f * er * er;
                });
        }
        if (step + 1 < 2 / BI) __syncthreads();        // the scratch is operand space again
    }
    if (over) F.flags[0] = 1;                         // an entry beyond the bound of a positive semi-definite matrix
    if (op == OP_M) {
        __syncthreads();
        store_partial(rsum, reinterpret_cast<float *>(smem), F.partial + ti * (ti + 1) / 2 + tj + half * F.ntri, lane, wave, tid, 4);
    }
}

// One launch per class of factors: NS = 4 (levels 4 or 5) and NS = 5 (levels 5 or 6).
template <int NS>
__global__ __launch_bounds__(256, 2) void digit_product_kernel(const FactorDev *__restrict__ fd, const FactorScal *__restrict__ fs,
                                                               const int *__restrict__ state, const uint2 *__restrict__ map, int total,
                                                               int op, int k, int degree)
{
    extern __shared__ __align__(16) unsigned char plane_smem[];
    const int w = xcd_tile(2 * total);
    if (w >= 2 * total) return;
    const uint2 tile = map[w >> 1];
    const int f = (int)tile.x, st = state[f];
    if (st != ST_RUN && !(st == ST_LAST && op == OP_SQ)) return;
    const FactorScal &S = fs[f];
    if (S.tier != TIER_DIGIT || S.ns != NS) return;
    const int ti = (int)(tile.y >> 16), tj = (int)(tile.y & 0xffffu), half = w & 1;
    if constexpr (NS == 4) {
        if (S.levels == 4) digit_tile<4, 4, 2>(fd[f], S, op, k, degree, ti, tj, half, plane_smem);
        else digit_tile<4, 5, 2>(fd[f], S, op, k, degree, ti, tj, half, plane_smem);
    } else {
        if (S.levels == 5) digit_tile<5, 5, 1>(fd[f], S, op, k, degree, ti, tj, half, plane_smem);
        else digit_tile<5, 6, 1>(fd[f], S, op, k, degree, ti, tj, half, plane_smem);
    }
}

template <int NS>
inline hipError_t launch_digit_product(const FactorDev *fd, const FactorScal *fs, const int *state, const uint2 *map, int total,
                                       int op, int k, int degree, hipStream_t stream)
{
    if (total <= 0) return hipSuccess;
    constexpr size_t lds = 2 * (size_t)PlaneLoader<2 * NS, NS == 4 ? 128 : 64, 64, 4>::STAGE;
    static_assert(lds >= 4 * (size_t)PLANE_SCRATCH_BYTES, "store scratch fits the stages");
    static bool configured[MAX_DEVICES] = {};
    if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(digit_product_kernel<NS>), lds, configured); e != hipSuccess) return e;
    const int per = (2 * total + NUM_XCD - 1) / NUM_XCD;
    profile_begin(300 + NS, stream);
    hipLaunchKernelGGL(digit_product_kernel<NS>, dim3(per * NUM_XCD), dim3(256), lds, stream, fd, fs, state, map, total, op, k, degree);
    profile_end(stream);
    return hipGetLastError();
}

}  // namespace asteria
