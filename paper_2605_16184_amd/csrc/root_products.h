// The products of the coupled root iteration on plane storage (planes.h): one kernel on pair planes (fp16
// matrix cores), one on digit planes (int8 matrix cores).  Every product is symmetric and has the form
//     C = k1 O1 + k2 O2 + g A B        (A, B, O1, O2, C symmetric, commuting)
// with per-factor coefficients that the control kernel has left on the device; only tiles on or below the
// diagonal are computed, their mirror images are stored with them.
#pragma once
#include <algorithm>
#include <type_traits>

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
inline int xcd_blocks(int total) { return (total + NUM_XCD - 1) / NUM_XCD * NUM_XCD; }

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
// C of one tile per workgroup of WGM x WGN wavefronts; a wavefront owns MI x NJ MFMA blocks of 16 x 16, slabs of 32 k, ST
// stages of LDS.  Three fp16 products per block and slab (lo hi, hi lo, hi hi: both operands to 2^-22) start from zero
// and the block's fp32 sum takes them in one addition: one rounding at full size per 32 k.
//
// Of a pair plane only the tiles on and below the diagonal (tiles of the launch's size, whole on the diagonal) are
// written and read.  An operand row beyond its diagonal tile comes from the column that mirrors it: a slab is then 32
// rows of the plane as they lie in memory, and the MFMA operands come out of LDS through transposed reads.
//
// Bound by power and by HBM: operands that toggle hold the clock at 1.7 GHz, and a product of n = 1024 has 80 flop per
// byte of its matrices and fp16 pass.  Hence one triangle, and tiles of 256 x 256 on 8 wavefronts (64 x 128 each), which read
// two thirds of the LDS bytes and half of the L2 bytes of 128 x 128 on 4.
//   - Operands go from memory to LDS without registers.
//   - The barrier between two slabs comes before the last column block of a slab: the next slab's first operands are
//     read behind those products, and its loads are spread between them.
//   - The linear term's loads are one block ahead of the arithmetic; a block goes through 4 KiB of LDS once and leaves
//     in whole lines.
// Measured, single product of the kind E2 (with the X update), against 128 x 128 tiles with whole planes and running sums
// for either kind of term: 600 of n = 1024 2.20 (4.56) ms, 2.50 (5.28) before; 8 of n = 4096 1.53 (3.00), 1.87 (3.49); 900 of
// n = 768 1.64 (3.41), 1.89 (4.24).  Of the 2.20 ms the K loop is 1.71 (1.27 PFLOP/s issued, 3900 cycles a slab for 3072 of
// MFMA), loading the linear term 0.14, storing 0.2.  Error of the root that does not commute with A, log-spaced spectrum,
// eps = 1e-6, n = 2048: 2.8e-4, 4.5e-4 before.
template <int WGM, int WGN, int MI, int NJ, int ST>
struct PairShape {
    static constexpr int NW = WGM * WGN, TM = 16 * MI * WGM, TN = 16 * NJ * WGN;
    static constexpr int NI = (TM + TN) / (8 * NW);          // load instructions of a wavefront per slab
    static constexpr int H = NI >= 8 ? NI / 2 : NI;           // ... of these issued behind the last column block of a slab
    static constexpr uint32_t STAGE = (uint32_t)TM * 128u;    // bytes per operand and stage
    static constexpr int KR = 256 / TM;                       // rows of a transposed slab per load instruction
    static constexpr uint32_t SCRATCH = 2u * ST * STAGE;
    static constexpr size_t LDS = SCRATCH + NW * 4096u;
    static_assert(TM == TN && NW % 2 == 0 && (NI & 1) == 0 && (TM / (NW / 2)) == 8 * NI, "half of the wavefronts load A, half B");
    static_assert(MI % 2 == 0 && NJ % 2 == 0 && (ST & (ST - 1)) == 0 && KR * TM == 256, "blocks of 32 x 32; stages by mask");
};

// Whether the 32 x 32 block at (br, bc) is one that a launch computes: on or below the diagonal and not wholly outside.  Nothing
// is read for the others either: what lies beyond row n - 1 of the caller's X is not his matrix.
__host__ __device__ inline bool pair_block_live(int br, int bc, int n) { return br >= bc && br < n && bc < n; }

// Element v = 4 (2 u + w) + e of a lane in a 32 x 32 block: row 16 u + lane % 16, column 16 w + 4 (lane / 16) + e
__host__ __device__ inline int pair_elem_row(int br, int v, int lane) { return br + 16 * (v >> 3) + (lane & 15); }
__host__ __device__ inline int pair_elem_col(int bc, int v, int lane) { return bc + 16 * ((v >> 2) & 1) + 4 * (lane >> 4) + (v & 3); }

// Whether X is read 4 columns at a time in a block at column bc (rows kept inside the matrix): all of its columns are the matrix's
__host__ __device__ inline bool pair_x_whole(int bc, int n, bool xvec) { return xvec && bc + 32 <= n; }

// two values (scaled) -> their hi terms and their lo terms, both rounded to nearest
__device__ __forceinline__ void pair_words2(float a, float b, uint32_t &hi, uint32_t &lo)
{
    typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
    const _Float16 ha = (_Float16)a, hb = (_Float16)b;
    hi = __builtin_bit_cast(uint32_t, (f16x2_t){ha, hb});
    lo = __builtin_bit_cast(uint32_t, (f16x2_t){(_Float16)(a - (float)ha), (_Float16)(b - (float)hb)});
}

template <int WGM, int WGN, int MI, int NJ, int ST>
__global__ __launch_bounds__(64 * WGM * WGN, 2) void pair_product_kernel(const FactorDev *__restrict__ fd, const FactorScal *__restrict__ fs,
                                                              const int *__restrict__ state, const uint2 *__restrict__ map, int total,
                                                              int op0, int op1, int k, int degree)
{
    using SH = PairShape<WGM, WGN, MI, NJ, ST>;
    constexpr int NW = SH::NW, NI = SH::NI, H = SH::H, TM = SH::TM, KR = SH::KR;
    constexpr uint32_t STAGE = SH::STAGE, KROW = (uint32_t)TM * 4u;      // bytes of a row of a transposed slab
    typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
    typedef _Float16 f16x4_t __attribute__((ext_vector_type(4)));
    typedef short s16x4_t __attribute__((ext_vector_type(4)));
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
    const FactorDev &F = fd[f];
    const int tier = S.tier, st0 = state[f];
    if (op != OP_X && tier != TIER_PAIR) return;
    const bool makes_e = op == OP_SQ || op == OP_SQ3 || op == OP_CUBE;
    const int st = __builtin_amdgcn_readfirstlane(makes_e ? st0 : state_after_test(F, S, st0));
    if (st != ST_RUN && !(st == ST_LAST && (makes_e || op == OP_X))) return;
    const int ti = (int)(tile.y >> 16), tj = (int)(tile.y & 0xffffu);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // position of the wavefront in the tile; of eight, those that share a SIMD (w, w + 4) have about the same work together in
    // a diagonal tile
    const int wm = NW == 8 ? (0x20103132 >> (4 * wave)) & 0xf : wave / WGN, wn = NW == 8 ? (0xB8 >> wave) & 1 : wave % WGN;
    const int n = F.n, rowb = F.rowb, p = k & 1, row0 = ti * TM, col0 = tj * TM, nk = plane_groups(n);
    const RootOperands o = root_operands(op, degree == 1);

    const char *O1 = nullptr, *O2 = nullptr;
    char *C = op == OP_X ? F.X[p ^ 1] : F.P[o.C];
    if (op != OP_X && o.O1 >= 0) O1 = F.P[o.O1];
    if (op != OP_X && o.O2 >= 0) O2 = F.P[o.O2];
    ASTERIA_GLOBAL float *X = (ASTERIA_GLOBAL float *)F.Xout;
    const int ldx = F.ldx;
    const bool xvec = (ldx & 3) == 0 && (reinterpret_cast<uintptr_t>(F.Xout) & 15u) == 0;
    // linear term of a block: 4 columns of a row, hi in [0 .. 1], lo in [2 .. 3]
    auto load_own = [&](const char *O, int br, int bc, int ln, uint32_t (&raw)[16]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const char *q = O + (size_t)min(br + 16 * u + (ln & 15), n - 1) * rowb + (min(bc, n - 1) >> 5) * 128 + (ln >> 4) * 8;
#pragma unroll
            for (int w = 0; w < 2; ++w) {
                const u32x2_t a = *(const ASTERIA_GLOBAL u32x2_t *)(q + w * 32), c = *(const ASTERIA_GLOBAL u32x2_t *)(q + w * 32 + 64);
                uint32_t *d = &raw[4 * (2 * u + w)];
                d[0] = a[0]; d[1] = a[1]; d[2] = c[0]; d[3] = c[1];
            }
        }
    };
    // fp32 X: its lower triangle until the last update, which completes the caller's matrix.  (On the diagonal the elements above it are
    // read with the others and not used.)
    auto load_x = [&](int br, int bc, int ln, uint32_t (&raw)[16]) __attribute__((always_inline)) {
        const bool whole = pair_x_whole(bc, n, xvec);
#pragma unroll
        for (int uw = 0; uw < 4; ++uw) {
            const int row = pair_elem_row(br, 4 * uw, ln), col = pair_elem_col(bc, 4 * uw, ln);
            const ASTERIA_GLOBAL float *x = X + (size_t)min(row, n - 1) * ldx + col;
            if (whole) {
                const u32x4 t = *(const ASTERIA_GLOBAL u32x4 *)x;
#pragma unroll
                for (int e = 0; e < 4; ++e) raw[4 * uw + e] = t[e];
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) raw[4 * uw + e] = row < n && row >= col + e ? __builtin_bit_cast(uint32_t, x[e]) : 0u;
            }
        }
    };
    uint32_t ahead[16];                               // linear term of the next block
    auto prefetch = [&](int br, int bc, int ln) __attribute__((always_inline)) {
        if (!pair_block_live(br, bc, n)) return;
        if (O1) load_own(O1, br, bc, ln, ahead);
        else if (op == OP_X) load_x(br, bc, ln, ahead);
    };
    // that of the first block before anything else, where there are registers to hold it through the K loop: a product of a small
    // matrix is little more than what it waits for (roots of 400 of n = 64: 670 us, 688 with the load behind the loop)
    constexpr bool EARLY = TM < 256;
    const int rw = row0 + wm * 16 * MI, cw = col0 + wn * 16 * NJ;
    if (EARLY) prefetch(rw, cw, lane);

    // ---- memory -> LDS: half of the wavefronts bring rows of A, half of B
    const bool loads_b = wave >= NW / 2;
    const char *src = op == OP_X ? (loads_b ? F.P[degree == 1 ? 0 : 2] : F.X[p]) : F.P[loads_b ? o.B : o.A];
    const int panel = loads_b ? tj : ti, i0 = (wave % (NW / 2)) * NI;    // first of this wavefront's load instructions
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds, ldst = lds0 + (loads_b ? ST * STAGE : 0u) + (uint32_t)i0 * 1024u;
    // direct: an instruction brings 8 rows, lane / 8 the row, lane % 8 the position of a 16-byte chunk (swizzle of plane_swz).
    // Rows beyond the matrix read as zero through the bounds of the descriptor
    const i32x4 rs_d = buffer_rsrc(src + (size_t)panel * TM * rowb, (uint32_t)min(n - panel * TM, TM) * (uint32_t)rowb);
    const uint32_t lch0 = (uint32_t)((lane & 7) ^ (lane >> 4)) * 16u;
    // transposed: an instruction brings KR rows of the TM columns of this panel; pieces of 32 bytes swizzled by row so that
    // the 4 rows of a 16-lane group of a transposed read lie in distinct banks
    const i32x4 rs_t = buffer_rsrc(src + (size_t)panel * TM * 4, (uint32_t)n * (uint32_t)rowb - (uint32_t)panel * TM * 4u);
    const uint32_t tk = (uint32_t)(lane / (64 / KR));
    const uint32_t off_d = (uint32_t)(i0 * 8 + (lane >> 3)) * (uint32_t)rowb + lch0;
    const uint32_t off_t = (((uint32_t)(lane % (64 / KR)) * 16u) ^ ((tk | ((uint32_t)(i0 * KR) >> 1 & 4u)) << 5));
    const uint32_t row_t = tk * (uint32_t)rowb;
    const int direct_end = (panel + 1) * (TM / 32);            // slabs from here on are transposed
    // loads v0 .. v0 + cnt - 1 of slab s (beyond the end: slab nk - 1 again, never read)
    auto issue = [&](int s, int v0, int cnt) __attribute__((always_inline)) {
        const int slab = min(s, nk - 1);
        const uint32_t dst = ldst + ((uint32_t)s & (ST - 1)) * STAGE;
        // all ones: direct.  Selected by masks, not branched on: a branch would cut the schedule of the products
        uint32_t d = (uint32_t)__builtin_amdgcn_readfirstlane((slab - direct_end) >> 31);
        asm("" : "+s"(d));
        auto pick = [&](uint32_t x, uint32_t y) __attribute__((always_inline)) { return y ^ ((x ^ y) & d); };
        i32x4 rs;
#pragma unroll
        for (int e = 0; e < 4; ++e) rs[e] = (int)pick((uint32_t)rs_d[e], (uint32_t)rs_t[e]);
        uint32_t off = pick(off_d, off_t);
        asm volatile("" : "+v"(off));                 // (the offsets of all loads are not worth registers)
        const uint32_t first = pick((uint32_t)slab * 128u, (uint32_t)(slab * 32 + i0 * KR) * (uint32_t)rowb);
        const uint32_t row_step = pick(8u, (uint32_t)KR) * (uint32_t)rowb;
#pragma unroll
        for (int v = v0; v < v0 + cnt; ++v) {
            const uint32_t kl = (uint32_t)v * KR, sw = pick((v & 1) * 64u, ((kl & 3u) | ((kl >> 1) & 4u)) << 5);
            load_to_lds(rs, dst + v * 1024, (off ^ sw) + ((uint32_t)v * row_step + first) + (KR > 1 ? pick(0u, row_t) : 0u), 0u);
        }
    };
#pragma unroll
    for (int s = 0; s < ST - 1; ++s) issue(s, 0, NI);
    issue(ST - 1, 0, H);

    // ---- what the values of the blocks are made of: loaded and worked out while the operands are on their way
    float sA, sB, s1 = 1.0f, s2 = 1.0f, sC;
    if (op == OP_X) {
        sA = sC = S.x_scale; sB = degree == 1 ? PAIR_SCALE_M : PAIR_SCALE_E;
    } else {
        sA = pair_scale_of(op, o.A); sB = pair_scale_of(op, o.B);
        if (O1) s1 = pair_scale_of(op, o.O1);
        if (O2) s2 = pair_scale_of(op, o.O2);
        sC = pair_scale_of(op, o.C);
    }
    const RootProd pc = S.prod[op];
    const float k1 = uniform((float)(pc.own1 * (double)(sC / s1))), k2 = uniform((float)(pc.own2 * (double)(sC / s2)));
    const float kg = uniform((float)(pc.gam * (double)sC / ((double)sA * (double)sB)));
    const bool to_user = op == OP_X && st == ST_LAST;
    const bool first_x = k == 0 && (op == OP_SQ || op == OP_CUBE);    // X_1 = X_0 T_0, X_0 a multiple of I
    const float inv_c = uniform(1.0f / sC);
    const float x1a = S.x1a, x1e = uniform(-S.x1s * inv_c), inv_x = uniform(1.0f / S.x_scale);
    // the test before the last update, by the product that completes E
    const bool test = st == ST_LAST && S.q_limit > 0.0f && ((op == OP_SQ && degree == 2) || op == OP_CUBE);
    const float q1 = uniform(S.q[1] / s1), q2 = uniform(S.q[2] / s2), q3 = uniform(S.q[3] * inv_c), q0 = S.q[0];

    // ---- LDS -> registers -> products
    const int a_end = (ti + 1) * (TM / 32), b_end = (tj + 1) * (TM / 32);
    uint32_t fa_d, fb_d, fa_t, fb_t;
    {
        const int r16 = lane & 15, g16 = lane >> 4;
        const uint32_t d = lds0 + (uint32_t)r16 * 128u + (uint32_t)((g16 ^ ((r16 >> 1) & 7)) * 16);
        fa_d = d + (uint32_t)(wm * 16 * MI) * 128u; fb_d = d + ST * STAGE + (uint32_t)(wn * 16 * NJ) * 128u;
        // lane 4 e + q of a 16-lane group supplies the address of rows 4 q .. of k = 8 g16 + e
        const int e = r16 >> 2;
        const uint32_t t = lds0 + (uint32_t)(8 * g16 + e) * KROW + (uint32_t)((e | ((g16 & 1) << 2)) << 5) + (uint32_t)(r16 & 3) * 8u;
        const uint32_t ga = (uint32_t)(wm * MI / 2), gb = (uint32_t)(wn * NJ / 2);     // first group of 32 rows; its low bit is swizzled
        fa_t = (t ^ ((ga & 1u) << 7)) + (ga >> 1) * 256u; fb_t = (t ^ ((gb & 1u) << 7)) + (gb >> 1) * 256u + ST * STAGE;
    }
    // 16 rows of an operand, hi (term 0) or lo: 8 consecutive k per lane.  x: 16-row block of the wavefront
    auto frag_d = [](uint32_t base, int x, int term) __attribute__((always_inline)) {
        return *(const ASTERIA_LDS u32x4 *)(uintptr_t)((term ? base ^ 64u : base) + x * 2048);
    };
    auto frag_t = [](uint32_t base, int x, int term) __attribute__((always_inline)) {
        // piece of 32 bytes 4 (x / 2) + 2 term + x % 2, its low three bits swizzled
        const int g = 4 * (x >> 1) + 2 * term + (x & 1);
        const uint32_t a = (base ^ (uint32_t)((g & 7) << 5)) + (uint32_t)((g >> 3) * 256);
        const u32x2_t lo = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((ASTERIA_LDS s16x4_t *)(uintptr_t)a));
        const u32x2_t hi = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((ASTERIA_LDS s16x4_t *)(uintptr_t)(a + 4 * KROW)));
        return (u32x4){lo[0], lo[1], hi[0], hi[1]};
    };
    // D = B-rows x A-rows: a lane then holds 4 consecutive columns of one row of C
    auto mma = [](u32x4 a, u32x4 b, floatx4 c) __attribute__((always_inline)) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(pl_f16x8, b), __builtin_bit_cast(pl_f16x8, a), c, 0, 0, 0);
    };
    wait_lds_loads<(ST - 2) * NI + H>();
    __builtin_amdgcn_s_barrier();

    // The tile for a wavefront whose first JN column blocks are wanted.  A body per width instead of branches in the loop: the
    // accumulators stay in their registers
    auto body = [&](auto jnc) __attribute__((always_inline)) {
        constexpr int JN = decltype(jnc)::value, JA = JN ? JN : 1;
        floatx4 acc[MI][JA];
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < JA; ++j) acc[i][j] = (floatx4){0.0f, 0.0f, 0.0f, 0.0f};
        const floatx4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
        u32x4 ah[MI], al[MI], b[2][2];
        uint32_t so = 0;                              // stage of the slab being read
        auto read_a = [&](u32x4 (&d)[MI], int term, int kt) __attribute__((always_inline)) {
            if (kt < a_end) {
#pragma unroll
                for (int i = 0; i < MI; ++i) d[i] = frag_d(fa_d + so, i, term);
            } else {
#pragma unroll
                for (int i = 0; i < MI; ++i) d[i] = frag_t(fa_t + so, i, term);
            }
        };
        auto read_b0 = [&](u32x4 (&d)[2], int kt) __attribute__((always_inline)) {
            if (kt < b_end) { d[0] = frag_d(fb_d + so, 0, 0); d[1] = frag_d(fb_d + so, 0, 1); }
            else { d[0] = frag_t(fb_t + so, 0, 0); d[1] = frag_t(fb_t + so, 0, 1); }
        };
        // the next slab has landed and everyone has read this one
        auto turn = [&](int kt) __attribute__((always_inline)) {
            wait_lds_loads<(ST - 2) * NI>();
            __builtin_amdgcn_s_barrier();
            so = ((uint32_t)(kt + 1) & (ST - 1)) * STAGE;
        };
        // AT, BT: the slab's rows of A, of B come from columns.  The next slab is read as if it were of the same kind: whoever
        // changes the kind reads again
        auto slab = [&](int kt, auto atc, auto btc) __attribute__((always_inline)) {
            constexpr bool AT = decltype(atc)::value, BT = decltype(btc)::value;
            auto next_a = [&](u32x4 (&d)[MI], int term) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < MI; ++i) d[i] = AT ? frag_t(fa_t + so, i, term) : frag_d(fa_d + so, i, term);
            };
            // the sums of a column block are taken while the next one is multiplied
            floatx4 t[2][MI];
#pragma unroll
            for (int j = 0; j < JN; ++j) {
                const int q = j & 1;
                const bool end = j + 1 == JN;
                if (!end) {
                    b[q ^ 1][0] = BT ? frag_t(fb_t + so, j + 1, 0) : frag_d(fb_d + so, j + 1, 0);
                    b[q ^ 1][1] = BT ? frag_t(fb_t + so, j + 1, 1) : frag_d(fb_d + so, j + 1, 1);
                } else {
                    turn(kt);
                    b[q ^ 1][0] = BT ? frag_t(fb_t + so, 0, 0) : frag_d(fb_d + so, 0, 0);
                    b[q ^ 1][1] = BT ? frag_t(fb_t + so, 0, 1) : frag_d(fb_d + so, 0, 1);
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int i = 0; i < MI; ++i) t[q][i] = mma(al[i], b[q][0], zero);
                if (end) { __builtin_amdgcn_sched_barrier(0); next_a(al, 1); issue(kt + ST, 0, H / 2); }
                if (H < NI && j == 0) { __builtin_amdgcn_sched_barrier(0); issue(kt + ST - 1, H, (NI - H) / 2); }
#pragma unroll
                for (int i = 0; i < MI; ++i) t[q][i] = mma(ah[i], b[q][1], t[q][i]);
                if (end) { __builtin_amdgcn_sched_barrier(0); issue(kt + ST, H / 2, H - H / 2); }
                if (H < NI && j == 0) { __builtin_amdgcn_sched_barrier(0); issue(kt + ST - 1, H + (NI - H) / 2, NI - H - (NI - H) / 2); }
#pragma unroll
                for (int i = 0; i < MI; ++i) t[q][i] = mma(ah[i], b[q][0], t[q][i]);
                if (j > 0)
#pragma unroll
                    for (int i = 0; i < MI; ++i) acc[i][j - 1] += t[q ^ 1][i];
                __builtin_amdgcn_sched_barrier(0);
            }
            next_a(ah, 0);
#pragma unroll
            for (int i = 0; i < MI; ++i) acc[i][JA - 1] += t[(JA - 1) & 1][i];
        };
        if constexpr (JN > 0) {
            auto read_all = [&](int kt) __attribute__((always_inline)) { read_a(al, 1, kt); read_a(ah, 0, kt); read_b0(b[0], kt); };
            read_all(0);
            int kt = 0;
            for (const int end = min(b_end, nk); kt < end; ++kt) slab(kt, std::false_type{}, std::false_type{});
            if (JN == NJ && a_end > b_end) {           // (a narrower body belongs to a diagonal tile)
                read_all(kt);
                for (const int end = min(a_end, nk); kt < end; ++kt) slab(kt, std::false_type{}, std::true_type{});
            }
            if (kt < nk) {
                read_all(kt);
                for (; kt < nk; ++kt) slab(kt, std::true_type{}, std::true_type{});
            }
        } else {
            for (int kt = 0; kt < nk; ++kt) {
                if (H < NI) issue(kt + ST - 1, H, NI - H);
                turn(kt);
                issue(kt + ST, 0, H);
            }
        }

        // ---- the block's value and its planes; in a diagonal tile its mirror image too
        float rsum = 0.0f;
        // The lane's part of every address is made anew for every block, not kept through the K loop.
        int ln = lane;
        asm volatile("" : "+v"(ln));
        int r16 = ln & 15, g16 = ln >> 4;
        ASTERIA_LDS char *ws = lds + SH::SCRATCH + wave * 4096;
        auto row_of = [&](int br, int v) { return pair_elem_row(br, v, ln); };
        auto col_of = [&](int bc, int v) { return pair_elem_col(bc, v, ln); };
        auto own_value = [&](const uint32_t (&raw)[16], int v) __attribute__((always_inline)) {
            const uint32_t *d = &raw[v & ~3];
            const f16x4_t a = __builtin_bit_cast(f16x4_t, (u32x2_t){d[0], d[1]}), c = __builtin_bit_cast(f16x4_t, (u32x2_t){d[2], d[3]});
            return (float)a[v & 3] + (float)c[v & 3];
        };
        auto store_x = [&](int br, int bc, const float (&x)[16], float c) __attribute__((always_inline)) {
#pragma unroll
            for (int uw = 0; uw < 4; ++uw) {
                const int row = row_of(br, 4 * uw), col = col_of(bc, 4 * uw);
                ASTERIA_GLOBAL float *d = X + (size_t)row * ldx + col;
                if (row >= n) continue;
                if (br > bc && xvec) *(ASTERIA_GLOBAL floatx4 *)d = (floatx4){x[4 * uw] * c, x[4 * uw + 1] * c, x[4 * uw + 2] * c, x[4 * uw + 3] * c};
                else
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (row >= col + e) d[e] = x[4 * uw + e] * c;
            }
        };
        // Planes of a block through the scratch, one row of the block per 128 bytes: [32 hi][32 lo], chunks swizzled by row.  Elements
        // beyond n are zero.  On the diagonal the upper triangle is taken from the lower one: every element from the block or from its
        // mirror image, by row and column.  (Written there element by element, up to 64 stores of 2 bytes a lane, it lay on the
        // critical path of small factors.  Roots of 400 of n = 64: 688 us so, 715 then.)
        auto store_block = [&](char *D, int br, int bc, const float (&val)[16]) __attribute__((always_inline)) {
            const bool diag = br == bc;
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int w = 0; w < 2; ++w) {
                    const float *q = &val[4 * (2 * u + w)];
                    uint32_t h0, h1, l0, l1;
                    pair_words2(q[0], q[1], h0, l0);
                    pair_words2(q[2], q[3], h1, l1);
                    const int r = 16 * u + r16, ch = 2 * w + (g16 >> 1);
                    ASTERIA_LDS char *d = ws + r * 128 + (g16 & 1) * 8;
                    *(ASTERIA_LDS u32x2_t *)(d + (ch ^ (r & 7)) * 16) = (u32x2_t){h0, h1};
                    *(ASTERIA_LDS u32x2_t *)(d + ((4 + ch) ^ (r & 7)) * 16) = (u32x2_t){l0, l1};
                }
            __builtin_amdgcn_wave_barrier();
            if (!diag)
#pragma unroll
                for (int q = 0; q < 4; ++q) {                   // whole lines of 8 rows
                    const int r = q * 8 + (ln >> 3), ch = ln & 7;
                    const u32x4 t = *(const ASTERIA_LDS u32x4 *)(ws + r * 128 + ((ch ^ (r & 7)) * 16));
                    if (br + r < n) *(ASTERIA_GLOBAL u32x4 *)(D + (size_t)(br + r) * rowb + (bc >> 5) * 128 + ch * 16) = t;
                }
            if (ti == tj) {
                // columns 16 (q & 1) .. of the block, hi or lo, as rows of the mirror image: a group of 16 lanes brings 8 rows of
                // the block; lane 4 e + i of it supplies the address of columns 4 i .. of row e, lane j receives column j
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int rh = q & 1, term = q >> 1, cl = 16 * rh + r16;
                    u32x2_t t[2];
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const int r = 4 * (2 * g16 + u) + (r16 >> 2), ch = term * 4 + rh * 2 + ((r16 & 3) >> 1);
                        t[u] = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                   (ASTERIA_LDS s16x4_t *)(ws + r * 128 + ((ch ^ (r & 7)) * 16) + (r16 & 1) * 8)));
                    }
                    u32x4 out = {t[0][0], t[0][1], t[1][0], t[1][1]};
                    if (diag) {
                        const u32x4 own = *(const ASTERIA_LDS u32x4 *)(ws + cl * 128 + (((term * 4 + g16) ^ (cl & 7)) * 16));
                        const int below = cl + 1 - 8 * g16;           // of the 8 columns from 8 g16 on, those on and below the diagonal
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const uint32_t m = below >= 2 * e + 2 ? ~0u : (below == 2 * e + 1 ? 0xffffu : 0u);
                            out[e] ^= (out[e] ^ own[e]) & m;
                        }
                    }
                    if (bc + cl < n) *(ASTERIA_GLOBAL u32x4 *)(D + (size_t)(bc + cl) * rowb + (br >> 5) * 128 + term * 64 + g16 * 16) = out;
                }
            }
            __builtin_amdgcn_wave_barrier();
        };
        constexpr int JB = JA / 2 ? JA / 2 : 1, NB = (MI / 2) * (JN / 2);
        auto block_row = [&](int q) { return rw + (q / JB) * 32; };
        auto block_col = [&](int q) { return cw + (q % JB) * 32; };
        if constexpr (NB > 0 && !EARLY) prefetch(rw, cw, ln);
        // one copy of the code for all blocks: only taking the sums out of their registers differs
#pragma unroll 1
        for (int q = 0; q < NB; ++q) {
            const int br = block_row(q), bc = block_col(q);
            asm volatile("" : "+v"(ln));
            r16 = ln & 15; g16 = ln >> 4;
            uint32_t raw[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) raw[v] = ahead[v];
            if (O2) load_own(O2, br, bc, ln, ahead);      // (a second linear term takes the place of the block ahead)
            else if (q + 1 < NB) prefetch(block_row(q + 1), block_col(q + 1), ln);
            if (!pair_block_live(br, bc, n)) {
                if (O2 && q + 1 < NB) prefetch(block_row(q + 1), block_col(q + 1), ln);
                continue;
            }
            float val[16];
#pragma unroll
            for (int z = 0; z < NB; ++z)
                if (q == z) {
                    asm volatile("");                 // a branch, not selects
#pragma unroll
                    for (int v = 0; v < 16; ++v) val[v] = kg * acc[2 * (z / JB) + (v >> 3)][2 * (z % JB) + ((v >> 2) & 1)][v & 3];
                }
            const bool diag = br == bc, inside = !diag && br + 32 <= n;
            // sums over the symmetric matrix: an element below the diagonal counts twice
            auto add_sum = [&](int v, float x) __attribute__((always_inline)) {
                const int row = row_of(br, v), col = col_of(bc, v);
                const float y = inside || (row < n && row >= col) ? x : 0.0f;
                rsum += inside || row != col ? 2.0f * y * y : y * y;
            };
            auto on_diag = [&](int v) { return row_of(br, v) == col_of(bc, v); };
            if (test) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float o1 = own_value(raw, v), o2 = O2 ? own_value(ahead, v) : 0.0f;
                    val[v] += k1 * o1 + (O2 ? k2 * o2 : 0.0f);
                    add_sum(v, q1 * o1 + (O2 ? q2 * o2 : 0.0f) + q3 * val[v] + (on_diag(v) ? q0 : 0.0f));
                }
            } else if (O1) {
#pragma unroll
                for (int v = 0; v < 16; ++v) val[v] += k1 * own_value(raw, v);
                if (O2)
#pragma unroll
                    for (int v = 0; v < 16; ++v) val[v] += k2 * own_value(ahead, v);
            } else if (op == OP_X) {
#pragma unroll
                for (int v = 0; v < 16; ++v) val[v] += k1 * __builtin_bit_cast(float, raw[v]);
            }
            if (O2 && q + 1 < NB) prefetch(block_row(q + 1), block_col(q + 1), ln);
            if (op == OP_M)
#pragma unroll
                for (int v = 0; v < 16; ++v) add_sum(v, val[v] * inv_c - (on_diag(v) ? 1.0f : 0.0f));
            if (op == OP_X) {
                store_x(br, bc, val, inv_c);
                if (to_user) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int row = row_of(br, v), col = col_of(bc, v);
                        if (row < n && row > col) X[(size_t)col * ldx + row] = val[v] * inv_c;
                    }
                    continue;
                }
            }
            if (br + 32 > n) {
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (row_of(br, v) >= n || col_of(bc, v) >= n) val[v] = 0.0f;
            }
            store_block(C, br, bc, val);
            if (first_x) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = row_of(br, v), col = col_of(bc, v);
                    val[v] = x1e * val[v] + (row == col && row < n ? x1a : 0.0f);
                }
                store_x(br, bc, val, inv_x);
                store_block(F.X[1], br, bc, val);
            }
        }
        if (op == OP_M || test) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) rsum += __shfl_xor(rsum, off, 64);
            if (lane == 0) *(ASTERIA_LDS float *)ws = rsum;
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            if (tid == 0) {
                float sum = 0.0f;
#pragma unroll
                for (int w = 0; w < NW; ++w) sum += *(const ASTERIA_LDS float *)(lds + SH::SCRATCH + w * 4096);
                (test ? F.qpart : F.partial)[ti * (ti + 1) / 2 + tj] = sum;
            }
        }
    };
    // column blocks of this wavefront with something on or below the diagonal and inside the matrix
    const int c = rw >= n ? 0 : min(ti == tj ? rw + 16 * MI : n, n) - cw;
    if (c <= 0) body(std::integral_constant<int, 0>{});
    else if (NJ == 8 && c <= 64) body(std::integral_constant<int, NJ == 8 ? 4 : NJ>{});
    else body(std::integral_constant<int, NJ>{});
    wait_lds_loads<0>();                              // nothing may land in LDS that is no longer this workgroup's
}

template <int WGM, int WGN, int MI, int NJ, int ST>
inline hipError_t launch_pair_product(const FactorDev *fd, const FactorScal *fs, const int *state, const uint2 *map, int total,
                                      int op0, int op1, int k, int degree, hipStream_t stream)
{
    if (total <= 0) return hipSuccess;
    using SH = PairShape<WGM, WGN, MI, NJ, ST>;
    auto kern = pair_product_kernel<WGM, WGN, MI, NJ, ST>;
    static bool configured[MAX_DEVICES] = {};
    if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kern), SH::LDS, configured); e != hipSuccess) return e;
    profile_begin(224, stream);
    hipLaunchKernelGGL(kern, dim3(xcd_blocks(op1 >= 0 ? 2 * total : total)), dim3(64 * SH::NW), SH::LDS, stream, fd, fs, state, map, total, op0, op1, k, degree);
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
// A workgroup of 2 x 2 wavefronts of 64 x 32 (two 32 x 32 MFMA blocks, L level accumulators each) computes one 128 x 64
// half of a tile, slabs of 32 k, two LDS stages of 24 (NS = 4) or 30 KiB: two workgroups per CU, so that one multiplies
// while the other assembles and stores.  In a slab the lower digits of A come first; the products of its top digit, most of
// all, cover the turn to the next slab.  Addresses and uniform factors of the epilogue are kept out of vector registers: nothing
// spills at four digits; at five, where 192 registers are sums at L = 6, 40 do (136 bytes of scratch a lane).
// Where at most 64 rows are left (BI = 1) a wavefront takes 32 of them: the epilogue of a block, an fp64 sum per level and element,
// is longer than its products there.  A product of 226 factors of n = 64, (5, 6): 14.0 us, 20.1 with half of the wavefronts taking 64
// rows each.
// Measured, kind E2: 8 of n = 4096 (5, 6) 4.24 ms = 2540 TOP/s issued, the matrix pipe full at the 1.75 GHz that power
// leaves (5.87 before, of which 1.1 went with the order of the tiles); 300 of n = 1024 (4, 4) 1.84 ms, 2.07 before, the
// epilogue a fifth of it; (5, 6) 3.22, 3.45 before.
// lower: 0 or 1 where a workgroup takes 64 rows of the half (BI = 1), -1 otherwise
template <int NS, int L, int BI>
__device__ __forceinline__ void digit_tile(const FactorDev &F, const FactorScal &S, int op, int k, int degree, int ti, int tj, int half,
                                           int lower, unsigned char *smem)
{
    constexpr int CPR = 2 * NS, ROWL = CPR * 16, RB = 64 * BI;
    using Loader = PlaneLoader<CPR, RB, 64, 4>;
    ASTERIA_LDS char *lds = (ASTERIA_LDS char *)smem;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1, r = lane & 31, h = lane >> 5;
    const int n = F.n, row0 = ti * 128 + (lower > 0 ? 64 : 0), col0 = tj * 128 + half * 64;
    if (col0 >= n || row0 >= n || (lower >= 0 && col0 > row0)) return;   // nothing to store; its partial sum was cleared when it was last read
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
    const double c1 = uniform(pc.own1 * qo), cg = uniform(pc.gam * qab);
    const double inv_q = uniform(ldexp(1.0, -S.dexp[op == OP_M ? 4 : o.C]));   // exponent slot 4: the next M
    const bool to_digits = !(op == OP_M && S.handover);
    // E feeds the X update as pair planes too (k > 0); so does M where T is linear or where the fp16 tier takes over
    const bool to_pair = (op == OP_SQ && k > 0) || (op == OP_M && (S.handover || S.pair_m));
    const bool first_x = op == OP_SQ && k == 0;       // X_1 = X_0 T_0, X_0 a multiple of I
    const double pe = uniform(first_x ? -(double)S.x1s : (op == OP_M ? (double)PAIR_SCALE_M : (double)PAIR_SCALE_E));
    const double pd = uniform(first_x ? (double)S.x1a : 0.0), inv_x = uniform(1.0 / (double)S.x_scale);
    float rsum = 0.0f;
    bool over = false;
    Loader ld;
    ld.init(digits_of(o.A), digits_of(o.B), rowb, n, row0, col0, wave, lane);
    i32x16 acc[L][BI];
#pragma unroll
    for (int l = 0; l < L; ++l)
#pragma unroll
        for (int i = 0; i < BI; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[l][i][v] = 0;
    // this wavefront's part lies above the diagonal or beyond the last row
    const bool above = row0 + (wm + 1) * 32 * BI - 1 < col0 + wn * 32 || row0 + wm * 32 * BI >= n;
    // address of digit 0; digit s lies 2 s chunks on, which the swizzle of 8 chunks makes an exclusive or
    uint32_t pa = lds0 + (uint32_t)(wm * 32 * BI + r) * ROWL + (uint32_t)((h ^ sw) * 16);
    uint32_t pb = lds0 + (uint32_t)(RB + wn * 32 + r) * ROWL + (uint32_t)((h ^ sw) * 16);
    auto digit = [](uint32_t p, int s, int off) __attribute__((always_inline)) {
        return *(const ASTERIA_LDS i32x4 *)(uintptr_t)((CPR == 8 ? (p ^ (uint32_t)(32 * s)) : p + 32 * s) + off);
    };
    i32x4 da[2][BI], db[NS];
    auto read_a = [&](int s) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < BI; ++i) da[s & 1][i] = digit(pa, s, i * 32 * ROWL);
    };
    // the products of digit s of A; consecutive ones write different accumulators
    auto times = [&](int s, int t) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < BI; ++i) acc[s + t][i] = __builtin_amdgcn_mfma_i32_32x32x32_i8(da[s & 1][i], db[t], acc[s + t][i], 0, 0, 0);
    };
    ld.issue(lds0, 0);
    ld.issue(lds0 + Loader::STAGE, min(1, last));
    wait_lds_loads<0>();
    __builtin_amdgcn_s_barrier();
    uint32_t cur = 0;
    if (above) {
        for (int kt = 0; kt < nk; ++kt) {
            wait_lds_loads<0>();
            __builtin_amdgcn_s_barrier();
            ld.issue(lds0 + cur, min(kt + 2, last));
            cur ^= (uint32_t)Loader::STAGE;
        }
    } else {
#pragma unroll
        for (int t = 0; t < NS; ++t) db[t] = digit(pb, t, 0);
        read_a(NS - 1);
        for (int kt = 0; kt < nk; ++kt) {
            // lowest digits of A first: the many products of its top digit, whose operands are all there, cover the turn
            // to the next slab, whose B takes the place of this one's digit by digit
#pragma unroll
            for (int s = NS - 1; s > 0; --s) {
                read_a(s - 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int t = 0; t < NS; ++t)
                    if (s + t < L) times(s, t);
                __builtin_amdgcn_sched_barrier(0);
            }
            wait_lds_loads<0>();                  // the next slab has landed ...
            __builtin_amdgcn_s_barrier();         // ... and everyone has read this one
            const uint32_t step = cur ? 0u - (uint32_t)Loader::STAGE : (uint32_t)Loader::STAGE;
            pa += step; pb += step;
#pragma unroll
            for (int t = 0; t < NS; ++t) {
                times(0, t);
                __builtin_amdgcn_sched_barrier(0);
                db[t] = digit(pb, t, 0);
                if (t == 0) ld.issue_part(lds0 + cur, min(kt + 2, last), 0, Loader::NI / 2);
                if (t == 1) ld.issue_part(lds0 + cur, min(kt + 2, last), Loader::NI / 2, Loader::NI);
                __builtin_amdgcn_sched_barrier(0);
            }
            read_a(NS - 1);
            cur ^= (uint32_t)Loader::STAGE;
        }
    }
    wait_lds_loads<0>();
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int i = 0; i < BI; ++i) {
        const int br = row0 + (wm * BI + i) * 32, bc = col0 + wn * 32;
        if (br < bc || br >= n || bc >= n) continue;
        int ln = lane;
        asm volatile("" : "+v"(ln));            // addresses are made here, not kept through the K loop
        const int r = ln & 31, h = ln >> 5;
        const int col = bc + r;
        const char *own = digits_of(o.O1) + (size_t)min(col, n - 1) * rowb + (br >> 5) * (32 * NS) + 16 * h;
        // calls use(v, row, value) for the block's elements; used once per output format (the second time
        // the own digits come from L1: cheaper than holding both formats in registers)
        auto values = [&](auto use) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                double ov[2][4];
                load_digit_groups<NS>(own, q, ov);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int g = q + 2 * (e >> 2), v = 4 * g + (e & 3), row = br + 8 * g + 4 * h + (e & 3);
                    double t = (double)acc[0][i][v];
#pragma unroll
                    for (int l = 1; l < L; ++l) t = t * 256.0 + (double)acc[l][i][v];
                    const double val = c1 * ov[e >> 2][e & 3] + cg * t;
                    use(v, row, (row < n && col < n) ? val : 0.0);
                }
            }
        };
        if (to_digits) {
            uint32_t wd[16], tp[4] = {0u, 0u, 0u, 0u};
            values([&](int v, int, double val) {
                uint32_t top;
                wd[v] = digit_word<NS>(val * inv_q, top, over);
                tp[v >> 2] |= top << (8 * (v & 3));
            });
            store_digit_block<NS>(digits_of(o.C), rowb, n, br, bc, wd, tp, ln, ws);
        }
        if (to_pair || first_x) {
            uint32_t pw[16];
            values([&](int v, int row, double val) {
                const double x = pe * val + (row == col ? pd : 0.0);
                pw[v] = (row < n && col < n) ? pair_word((float)x) : 0u;
                if (first_x && row < n && col < n && row >= col) F.Xout[(size_t)row * F.ldx + col] = (float)(x * inv_x);
            });
            store_pair_block(first_x ? F.X[1] : F.P[o.C], F.rowb, n, br, bc, pw, ln, ws);
        }
        if (op == OP_M)
            values([&](int, int row, double val) {
                const float er = (float)(val - (row == col ? 1.0 : 0.0));
                if (row < n && col < n && row >= col) rsum += row == col ? er * er : 2.0f * er * er;
            });
    }
    if (over) F.flags[0] = 1;                         // an entry beyond the bound of a positive semi-definite matrix
    if (op == OP_M) {
        // by tiles of 64 x 64, or by tile and half
        const int r64 = 2 * ti + max(lower, 0), at = lower >= 0 ? r64 * (r64 + 1) / 2 + 2 * tj + half : ti * (ti + 1) / 2 + tj + half * F.ntri;
        __syncthreads();
        store_partial(rsum, reinterpret_cast<float *>(smem), F.partial + at, lane, wave, tid, 4);
    }
}

// One half of a tile, or 64 rows of it (lower >= 0), by the digits of its factor (NS = 4: levels 4 or 5; NS = 5: levels 5 or 6).
template <int NS, bool QUARTER>
__device__ __forceinline__ void digit_half(const FactorDev &F, const FactorScal &S, int op, int k, int degree, uint2 tile, int half, int lower,
                                           unsigned char *smem)
{
    const int ti = (int)(tile.y >> 16), tj = (int)(tile.y & 0xffffu);
    auto run = [&](auto bi) __attribute__((always_inline)) {
        constexpr int BI = decltype(bi)::value;
        if (S.levels == NS) digit_tile<NS, NS, BI>(F, S, op, k, degree, ti, tj, half, lower, smem);
        else digit_tile<NS, NS + 1, BI>(F, S, op, k, degree, ti, tj, half, lower, smem);
    };
    if constexpr (QUARTER) run(std::integral_constant<int, 1>{});
    else if (F.n - ti * 128 <= 64) run(std::integral_constant<int, 1>{});
    else run(std::integral_constant<int, 2>{});
}

// One launch for factors of either number of digits (NS = 0) or one for each: figures where they are launched.  (NS = 0 spills what five
// digits do, NS = 4 nothing.)
// QUARTER: 64 x 64 per workgroup.  With few tiles the epilogue of two blocks one after the other is what a product waits for.  The line, us
// of the refresh, halves / quarters, by halves of tiles: figures beside PLANE_QUARTERS.
template <int NS, bool QUARTER>
__global__ __launch_bounds__(256, 2) void digit_product_kernel(const FactorDev *__restrict__ fd, const FactorScal *__restrict__ fs,
                                                               const int *__restrict__ state, const uint2 *__restrict__ map, int total,
                                                               int op, int k, int degree)
{
    constexpr int PARTS = QUARTER ? 4 : 2;
    extern __shared__ __align__(16) unsigned char plane_smem[];
    const int w = xcd_tile(PARTS * total);
    if (w >= PARTS * total) return;
    const uint2 tile = map[w / PARTS];
    const FactorScal &S = fs[tile.x];
    const int st = state[tile.x], ns = S.ns, half = w & 1, lower = QUARTER ? (w >> 1) & 1 : -1;
    if (S.tier != TIER_DIGIT || (st != ST_RUN && !(st == ST_LAST && op == OP_SQ))) return;
    if (NS == 4 || (NS == 0 && ns == 4)) { if (ns == 4) digit_half<4, QUARTER>(fd[tile.x], S, op, k, degree, tile, half, lower, plane_smem); }
    else if (ns == 5) digit_half<5, QUARTER>(fd[tile.x], S, op, k, degree, tile, half, lower, plane_smem);
}

constexpr size_t digit_lds(int ns) { return 2 * (size_t)(128 + 64) * (2 * ns) * 16; }     // two stages
static_assert(digit_lds(4) >= 4 * (size_t)PLANE_SCRATCH_BYTES, "store scratch fits the stages");

template <int NS, bool QUARTER = false>
inline hipError_t launch_digit_product(const FactorDev *fd, const FactorScal *fs, const int *state, const uint2 *map, int total,
                                       int op, int k, int degree, hipStream_t stream)
{
    if (total <= 0) return hipSuccess;
    constexpr size_t lds = digit_lds(NS == 0 ? 5 : NS);
    auto kern = digit_product_kernel<NS, QUARTER>;
    static bool configured[MAX_DEVICES] = {};
    if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kern), lds, configured); e != hipSuccess) return e;
    profile_begin(NS == 0 ? 304 : 300 + NS, stream);
    hipLaunchKernelGGL(kern, dim3(xcd_blocks((QUARTER ? 4 : 2) * total)), dim3(256), lds, stream, fd, fs, state, map, total, op, k, degree);
    profile_end(stream);
    return hipGetLastError();
}

}  // namespace asteria
