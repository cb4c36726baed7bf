// The plane path of asteria_inverse_root: the coupled iteration on plane storage (planes.h), taken under the
// fully automatic precision rules (relative eps, root 4, interval-adapted schedule, n <= 16384).
//
//   T = c0 I - E,  E = -(c1 M + c2 M^2 + c3 M^3)   degree 1, 2 or 3 by iteration (root_degrees)
//   E2 = 2 c0 E - E E      (T^2 = c0^2 I - E2)
//   W = c0^2 M - E2 M,  M' = c0^2 W - E2 W,  X' = c0 X - X E
//
// Neither T nor T^2 is stored, only their complements: those have the small diagonals of M (entries of
// a statistic with a decaying spectrum are of the size of its mean eigenvalue), which is what a fixed number of
// bits is measured against, and every product reads its linear term from an operand it has streamed anyway.
//
// While the bottom of M's spectrum is below ROOT_LOWP_FLOOR the chain runs on digit planes (int8 matrix cores,
// 32 or 40 bits against a uniform quantum), or, where the device finds 40 bits too few or the caller asked for
// it, on fp64 matrices;
// afterwards on pair planes.  X is kept in fp32, its lower triangle in the caller's matrix, and in pair planes as an
// operand of the next update.
#pragma once

namespace asteria {

// Errors allowed in the bottom `lo` of M's spectrum, relative to it (a quarter reaches the root there):
//   rounding of M to 2^-8NS of a bound d on its diagonal, an error matrix of norm below n^(1/2) 2^-8NS d;
//   the digit products beyond the kept levels, per entry (2 n^(1/2) of it in norm) about (pairs of the first
//   dropped level x n)^(1/2) 128^2 / 3 quanta of that level, for the products E2 W and (lifted by c0^2) E2 M,
//   against the bottom of M'.
// Measured against the same iteration on fp64 matrices (power law, rank 32 + noise, log-spaced over 12 and 16
// decades, two levels; n = 96 .. 1024): at these limits the root differs by less than 1.5e-4.
constexpr double DIGIT_ROUNDING = 9e-4;
constexpr double DIGIT_DROPPED = 3e-3;

__host__ __device__ inline double digit_rounding(int n, int ns, double d, double lo) { return sqrt((double)n) * ldexp(1.0, -8 * ns) * d / lo; }
// ranges: 2^ea, 2^eb bound the operands
__host__ __device__ inline double digit_dropped(int n, int ns, int levels, int ea, int eb)
{
    const int pairs = 2 * ns - 1 - levels;              // digit pairs s + t = levels
    if (pairs <= 0) return 0.0;
    return 2.0 * n * sqrt((double)pairs) * 5461.0 * ldexp(1.0, ea + eb - 2 * (8 * ns - 1) + 8 * (2 * (ns - 1) - levels));
}

// least e with x <= 2^e, x > 0
__device__ inline int ceil_log2(double x)
{
    int e;
    return frexp(x, &e) == 0.5 ? e - 1 : e;
}

// diagonal of M_0 above which a second prefix iteration of degree 2 is kept on digits: two fp16 terms are too
// coarse for entries of that size while the spectrum still reaches down to 4e-5
constexpr double DIGIT_WIDE_DIAG = 0.25;

struct PlaneControl {
    int k, degree, next_linear, prefix;   // prefix: iterations that may run on digits or in fp64
    int wide_next;                        // the next iteration has digit products (degree <= 2, inside the prefix)
    int digits_max;                       // 0, 4 or 5
    int final_pass;
    float stop_resid;
    // the host's T for this iteration, made for an interval a little wider than the one every factor of the common
    // eps arrives with: taken where it covers the factor's interval closely
    double lo, hi;
    RootPoly T;
    double *counters;                     // measurement aid (profile_i8_counters), or null
};

// Decide about iteration k of one factor and leave its coefficients (one thread).
__device__ inline void plane_advance(const FactorDev &F, FactorScal &S, int *state, float resid, const PlaneControl &c)
{
    int st = *state;
    S.resid = resid;
    const double lo0 = S.lo_d, hi0 = S.hi_d;
    const double dev = fmax(1.0 - lo0, hi0 - 1.0);
    // every |mu - 1| is at most the measured residual: tighten the predicted interval
    double lo = lo0, hi = hi0;
    const double rb = (double)resid * 1.001 + 1e-5;
    if (1.0 - rb > lo) lo = 1.0 - rb;
    if (1.0 + rb < hi) hi = 1.0 + rb;
    if (!(hi > lo)) { lo = 1.0 - rb; hi = 1.0 + rb; }
    const RootPoly T = (lo >= c.lo && hi <= c.hi && lo <= 1.001 * c.lo) ? c.T : root_poly(lo, hi, c.degree);
    // one more X update finishes the factor: see root_control_kernel for the three tests and what they rely on
    const bool consistent = (double)resid < 1.5 * sqrt((double)F.n) * dev + 2e-3;
    const double dev_next = fmax(1.0 - T.image.lo, T.image.hi - 1.0);
    const bool ends = resid < c.stop_resid || (consistent && dev < (double)ROOT_STOP_DEV) ||
                      (consistent && dev_next <= 4.0 * (double)ROOT_X_TOL);
    if (c.final_pass) {
        // eigenvalues in [0, hi] stay there, within 1 of 1; beyond that, one is negative
        S.info = resid > 1.1f * sqrtf((float)F.n) ? ASTERIA_INFO_NOT_PD : ASTERIA_INFO_NOT_CONVERGED;
        if (S.info == ASTERIA_INFO_NOT_PD) *state = ST_FAIL;
        return;
    }
    if (ends) st = ST_LAST;
    S.iters += 1;
    S.xloc = (st == ST_LAST && c.k > 0) ? 0 : 1;
    // T = a I - E; what M carries into the products where T is linear
    const double a = T.c[0], b = -T.c[1];
    const bool lin = c.degree == 1;
    S.prod[OP_SQ] = {b, 0.0, -T.c[2]};
    S.prod[OP_SQ3] = {0.0, 0.0, 1.0};
    S.prod[OP_CUBE] = {b, -T.c[2], -T.c[3]};
    S.prod[OP_E2] = lin ? RootProd{2.0 * a * b, 0.0, -b * b} : RootProd{2.0 * a, 0.0, -1.0};
    S.prod[OP_W] = {a * a, 0.0, -1.0};
    S.prod[OP_M] = {a * a, 0.0, -1.0};
    S.prod[OP_X] = lin ? RootProd{a, 0.0, -b} : RootProd{a, 0.0, -1.0};
    if (c.k == 0) {
        const double xs = sqrt(sqrt((double)S.scale)) * (double)S.x_scale;
        S.x1a = (float)(xs * a); S.x1s = (float)xs; S.x1b = (float)b;
    }
    // bounds on the diagonals (E <= b M, E2 <= 2 a E, W <= a^2 M, M' <= a^4 M in the order of symmetric
    // matrices, and every norm by the scalar map) and from them the quanta of the digits
    const double dm = S.dmax, de = lin ? dm : fmin(b * dm, a), de2 = fmin(2.0 * a * (lin ? b * dm : de), a * a);
    const double dw = fmin(a * a * dm, sqrt(T.image.hi * hi) * 1.001), dm1 = fmin(a * a * a * a * dm, T.image.hi * 1.001);
    // (beyond the prefix nothing runs on digits)
    int ge = 0, ge2 = 0, gw = 0, gm1 = 0, gm = 0;
    if (c.k < c.prefix) {
        ge = ceil_log2(de * 1.02); ge2 = ceil_log2(de2 * 1.02); gw = ceil_log2(dw * 1.02); gm1 = ceil_log2(dm1 * 1.02);
        gm = c.k > 0 && S.next_tier == TIER_DIGIT ? S.dexp[4] + 8 * S.ns - 1 : ceil_log2(dm * 1.02);      // the range the last M-update was stored with
    }
    // error of the dropped levels of E2 W and E2 M relative to the bottom of M'
    auto dropped = [&](int ns, int levels) {
        return (digit_dropped(F.n, ns, levels, ge2, gw) + a * a * digit_dropped(F.n, ns, levels, ge2, gm)) / T.image.lo;
    };
    // digits that are fine enough for this M: 4, 5, or 0
    auto digits = [&]() {
        if (c.digits_max >= 4 && digit_rounding(F.n, 4, dm, lo) <= DIGIT_ROUNDING && dropped(4, 5) <= DIGIT_DROPPED) return 4;
        return c.digits_max >= 5 && digit_rounding(F.n, 5, dm, lo) <= DIGIT_ROUNDING && dropped(5, 6) <= DIGIT_DROPPED ? 5 : 0;
    };
    S.from_f64 = 0;
    if (c.k == 0) {
        S.tier = TIER_PAIR;
        S.ns = 4;
        S.swapped = 0;
        if (c.prefix > 0 && lo < ROOT_LOWP_FLOOR) {
            const int ns = digits();
            S.tier = ns ? TIER_DIGIT : TIER_F64;
            if (ns) S.ns = ns;
        }
    } else {
        S.tier = S.next_tier;
        // the bottom of the spectrum has risen: where digits are enough now, the rest of the prefix runs on them (a
        // diagonal close to the largest eigenvalue at eps = 1e-8, 64 factors of n = 1024: 30.9 ms in fp64 throughout, 21.7)
        if (S.tier == TIER_F64 && c.k < c.prefix && c.degree <= 2)
            if (const int ns = digits()) {
                S.tier = TIER_DIGIT;
                S.ns = ns;
                S.from_f64 = S.swapped = 1;
            }
    }
    // The residual cannot tell one negative eigenvalue of M from n that deviate as they may, and after the last update
    // nothing is measured.  So the last product of E also sums the squares of the Chebyshev polynomial of its degree for
    // [lo, hi], which M, M^2 and E combine to: at most 1 for an eigenvalue inside, q(0)^2 or more for a negative one
    // (3900 in the last iteration of the schedule for eps = 1e-6).  Where they are more than n the iteration goes on:
    // eigenvalues that fell short of lo catch up, negative ones grow until they show.  A residual below 1 proves that
    // there are none.
    S.q_limit = 0.0f;
    if (ends && c.degree >= 2 && S.tier == TIER_PAIR && !(resid < 0.9f)) {
        const double m = 0.5 * (lo + hi), h = 0.5 * (hi - lo), x0 = -m / h;
        // powers of mu in T_2(x) = 2 x^2 - 1 or T_3(x) = 4 x^3 - 3 x, x = (mu - m) / h
        const bool cubic = c.degree == 3;
        const double p0 = cubic ? 4.0 * x0 * x0 * x0 - 3.0 * x0 : 2.0 * x0 * x0 - 1.0, p1 = (cubic ? 12.0 * x0 * x0 - 3.0 : 4.0 * x0) / h;
        const double p2 = (cubic ? 12.0 * x0 : 2.0) / (h * h), top = cubic ? 4.0 / (h * h * h) : p2;
        const double e = -top / T.c[c.degree];        // the leading power comes from E = -(c1 M + c2 M^2 + c3 M^3)
        S.q[0] = (float)p0; S.q[1] = (float)(p1 + e * T.c[1]); S.q[2] = cubic ? (float)(p2 + e * T.c[2]) : 0.0f; S.q[3] = (float)e;
        S.q_limit = 1.05f * (float)F.n + 10.0f;
    }
    if (S.tier == TIER_DIGIT) {
        const int bits = 8 * S.ns - 1;
        S.levels = dropped(S.ns, S.ns) <= (S.ns == 4 ? DIGIT_DROPPED : 0.2 * DIGIT_DROPPED) ? S.ns : S.ns + 1;
        S.dexp[0] = gm - bits; S.dexp[1] = ge2 - bits; S.dexp[2] = ge - bits; S.dexp[3] = gw - bits; S.dexp[4] = gm1 - bits;
    }
    if (c.counters) {
        // flops of this iteration's chain by where they run, of all pair products, and int8 operations issued
        const double one = (double)F.n * (double)F.n * (double)(F.n + 1);
        const double chain = one * (double)(c.degree - 1 + (st == ST_LAST ? 0 : 3)), x = c.k > 0 ? one : 0.0;
        const int passes = S.ns == 4 ? (S.levels == 4 ? 10 : 13) : (S.levels == 5 ? 15 : 19);
        if (S.tier == TIER_F64) atomicAdd(&c.counters[0], chain);
        if (S.tier == TIER_DIGIT) { atomicAdd(&c.counters[S.ns - 3], chain); atomicAdd(&c.counters[4], chain * passes); }
        atomicAdd(&c.counters[3], x + (S.tier == TIER_PAIR ? chain : 0.0));
    }
    const bool wide = c.wide_next && dm > DIGIT_WIDE_DIAG && c.k == 0;
    const bool to_pair = S.tier == TIER_PAIR || c.k + 1 >= c.prefix || (T.image.lo >= ROOT_LOWP_FLOOR && !wide);
    S.next_tier = to_pair ? TIER_PAIR : S.tier;
    S.handover = to_pair ? 1 : 0;
    S.pair_m = c.next_linear;
    S.dmax = dm1;
    S.lo_d = T.image.lo; S.hi_d = T.image.hi;
    *state = st;
}

// The order in which a launch takes the tiles of a factor: strips of 8 tile rows, columns within a strip.  The 64 half tiles
// that an XCD works on then read 8 + 4 panels of the operands instead of 1 + 32 (8 factors of n = 4096, digit products: 5.87 ms
// row by row, 4.9 in strips of 4, 4.76 of 8; n <= 1024 has one strip and does not care, nor do the pair products).
constexpr int TILE_STRIP = 8;
__device__ __forceinline__ void strip_decode(int t, int tiles, int &ti, int &tj)
{
    int r0 = 0;
    while (true) {
        const int h = min(TILE_STRIP, tiles - r0), full = h * (r0 + 1), all = full + h * (h - 1) / 2;
        if (t >= all) { t -= all; r0 += TILE_STRIP; continue; }
        if (t < full) { tj = t / h; ti = r0 + t % h; return; }
        t -= full;
        int c = 1;                                    // column r0 + c has the rows r0 + c .. r0 + h - 1
        while (t >= h - c) { t -= h - c; ++c; }
        tj = r0 + c; ti = r0 + c + t;
        return;
    }
}

// One workgroup per factor: scaling, start of the interval, and the decision about iteration 0.  lz_steps > 0: lambda_max comes from
// lanczos_cluster_kernel, whose workgroups may have given up.
__global__ __launch_bounds__(256) void plane_setup_kernel(const FactorDev *fd, FactorScal *fs, int *state, float margin, PlaneControl c,
                                                          uint2 *map128, uint2 *map_p, int pair_tile, float lz_tol2, int lz_steps)
{
    const int f = blockIdx.x;
    const FactorDev &F = fd[f];
    FactorScal &S = fs[f];
    if (lz_steps > 0 && S.pm_done == 0) lanczos_alone(F, S, lz_tol2, lz_steps);
    const int tid = threadIdx.x, n = F.n;
    __shared__ double red[3][4];
    // factor and tile of every workgroup of the tile-indexed launches
    for (int t = tid; t < F.ntri; t += 256) {
        int ti, tj;
        strip_decode(t, (n + 127) / 128, ti, tj);
        map128[F.tile_start + t] = make_uint2((unsigned)f, ((unsigned)ti << 16) | (unsigned)tj);
    }
    if (map_p) {
        const int nt = tri_tiles_of(n, pair_tile);
        for (int t = tid; t < nt; t += 256) {
            int ti, tj;
            strip_decode(t, (n + pair_tile - 1) / pair_tile, ti, tj);
            map_p[F.tile_start_p + t] = make_uint2((unsigned)f, ((unsigned)ti << 16) | (unsigned)tj);
        }
    }
    for (int t = tid; t < F.npart; t += 256) F.partial[t] = F.qpart[t] = 0.0f;
    double mx = 0.0, tr = 0.0;
    for (int i = tid; i < n; i += 256) {
        const double d = (double)F.A[F.a_packed ? packed_off(i, i) : (size_t)i * F.lda + i];
        mx = fmax(mx, d);
        tr += d;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) { mx = fmax(mx, __shfl_xor(mx, off, 64)); tr += __shfl_xor(tr, off, 64); }
    if ((tid & 63) == 0) { red[0][tid >> 6] = mx; red[1][tid >> 6] = tr; }
    __syncthreads();
    if (tid != 0) return;
    mx = fmax(fmax(red[0][0], red[0][1]), fmax(red[0][2], red[0][3]));
    tr = red[1][0] + red[1][1] + red[1][2] + red[1][3];
    const float lam = S.rho;
    S.lam = lam; S.iters = 0; S.xloc = 0; S.resid = 0.0f;
    F.flags[0] = 0;
    const float eps = F.eps_in * lam;
    S.eps = eps;
    const float denom = (1.0f + margin) * lam + eps;
    const bool ok = (lam == lam) && (lam >= 0.0f) && (lam < 3.0e38f) && (denom > 0.0f) && (denom < 3.0e38f) && (1.0f / denom < 3.0e38f);
    if (!ok) {
        S.scale = 0.0f; S.info = ASTERIA_INFO_NOT_PD; S.tier = TIER_PAIR;
        state[f] = ST_FAIL;
        return;
    }
    S.scale = 1.0f / denom;
    S.info = ASTERIA_INFO_OK;
    state[f] = ST_RUN;
    const double sc = (double)S.scale, e = (double)eps;
    // spectrum of M_0 = s (A + eps I): at most 1 by the scaling; at least eps s for a positive semi-definite A
    // (halved: round-off in the statistics may push eigenvalues slightly below 0)
    double lo = 0.5 * e / (double)denom;
    if (!(lo > 1e-12)) lo = 1e-12;
    // ||M_0 - I||_F bounds every |mu - 1|: a well-conditioned factor gets a much tighter interval
    const double f2 = S.fro2 + 2.0 * e * tr + n * e * e;
    double r2 = sc * sc * f2 - 2.0 * sc * (tr + n * e) + n;
    const double rs = r2 * (1.0 + 1e-3) + 1e-6 * n;                  // slack for the sums and for the fp32 scale
    if (rs > 0.0 && rs < 1.0) { const double l1 = 1.0 - sqrt(rs); if (l1 > lo) lo = l1; }
    // the difference of large terms stands in for a measured residual only where it can be one: a clearly negative
    // or non-finite value says nothing, and the interval is left as it is
    if (!(r2 >= -1e-6 * n) || !(r2 < 1e300)) r2 = (double)n * ROOT_TOP * ROOT_TOP;
    else if (r2 < 1e-6 * n) r2 = 1e-6 * n;
    // |X_k| <= xs (2 / lo)^(1/4) for every iterate (see root_setup_kernel): the fp16 terms of X are scaled by the
    // largest power of two that keeps this below 30000
    const double bound = sqrt(sqrt(sc)) * sqrt(sqrt(2.0 / lo));
    int ex = (int)floor(log2(30000.0 / bound));
    ex = ex < -60 ? -60 : (ex > 60 ? 60 : ex);
    S.x_scale = (float)ldexp(1.0, ex);
    S.dmax = fmax(sc * (mx + e), 1e-30);
    S.lo_d = lo; S.hi_d = ROOT_TOP;
    plane_advance(F, S, &state[f], (float)sqrt(r2), c);
}

// One wavefront per factor before iteration k >= 1 and after the last one.
__global__ __launch_bounds__(64) void plane_control_kernel(const FactorDev *fd, FactorScal *fs, int *state, PlaneControl c)
{
    const int f = blockIdx.x;
    const int st = state[f];
    if (st == ST_DONE || st == ST_FAIL) return;
    const FactorDev &F = fd[f];
    FactorScal &S = fs[f];
    if (state_after_test(F, S, st) == ST_LAST) {
        if (threadIdx.x == 0) {
            const bool over = F.flags[0] != 0;        // the last update's own products may still have run on digits
            if (over) S.info = ASTERIA_INFO_NOT_PD;
            state[f] = over ? ST_FAIL : ST_DONE;
        }
        return;
    }
    if (st == ST_LAST && threadIdx.x == 0) state[f] = ST_RUN;
    const float r2 = wave_total(F.partial, F.npart);
    for (int i = threadIdx.x; i < F.npart; i += 64) F.partial[i] = 0.0f;
    if (threadIdx.x != 0) return;
    if (!(r2 == r2) || !(r2 < 3.0e38f) || F.flags[0]) {
        S.info = ASTERIA_INFO_NOT_PD;
        S.resid = sqrtf(r2);
        state[f] = ST_FAIL;
        return;
    }
    plane_advance(F, S, &state[f], sqrtf(r2), c);
}

// M_0 = s (A + eps I) of one 128 x 128 tile and its mirror image in the storage of the factor's tier, and where T
// is linear X_1 = X_0 T_0.  A workgroup takes a 64 x 64 sub-tile of A (blockIdx.y) and its transposed position through LDS; a thread then
// owns 16 consecutive columns of a row.  HBM-bound: 4 bytes read, 4 or 5 written per element (8 or 9 with X_1).
__global__ __launch_bounds__(256) void plane_init_kernel(const FactorDev *fd, const FactorScal *fs, const int *state, const uint2 *map, int linear)
{
    const uint2 tile = map[blockIdx.x];
    const int f = (int)tile.x;
    if (state[f] == ST_FAIL) return;
    const FactorDev &F = fd[f];
    const FactorScal &S = fs[f];
    const int ti = (int)(tile.y >> 16), tj = (int)(tile.y & 0xffffu);
    const int n = F.n, lda = F.lda, tid = threadIdx.x;
    const double s = (double)S.scale, eps = (double)S.eps;
    const int tier = S.tier, ns = S.ns;
    const double inv_q = tier == TIER_DIGIT ? ldexp(1.0, -S.dexp[0]) : 0.0;
    const float x1a = S.x1a, x1e = S.x1s * S.x1b, inv_x = 1.0f / S.x_scale;
    const bool packed = F.a_packed != 0;
    const float *Ap = packed ? F.A + (size_t)(ti * (ti + 1) / 2 + tj) * PACK_T * PACK_T : nullptr;
    const bool vec = packed || ((lda & 3) == 0 && (reinterpret_cast<uintptr_t>(F.A) & 15u) == 0);
    __shared__ float Pw[64][65], Qw[64][65];
    bool over = false;
    // 16 columns c0 .. of row r of the symmetrised matrix: get(e) is the entry of A
    auto emit = [&](int r, int c0, auto get) {
        if (r >= n || c0 >= plane_groups(n) * 32) return;
        double m[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) m[e] = (c0 + e < n) ? s * (get(e) + (r == c0 + e ? eps : 0.0)) : 0.0;
        uint32_t w[16];
        const int grp = c0 >> 5, hf = (c0 >> 4) & 1;
        auto put_pair = [&](char *M) {
            char *d = M + (size_t)r * F.rowb + grp * 128 + hf * 32;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                u32x4 hi, lo;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    hi[e] = __builtin_amdgcn_perm(w[8 * q + 2 * e + 1], w[8 * q + 2 * e], 0x05040100u);
                    lo[e] = __builtin_amdgcn_perm(w[8 * q + 2 * e + 1], w[8 * q + 2 * e], 0x07060302u);
                }
                *(ASTERIA_GLOBAL u32x4 *)(d + q * 16) = hi;
                *(ASTERIA_GLOBAL u32x4 *)(d + 64 + q * 16) = lo;
            }
        };
        if (tier == TIER_DIGIT) {
            uint32_t t;
            u32x4 top = {0u, 0u, 0u, 0u};
            if (ns == 4) {
#pragma unroll
                for (int e = 0; e < 16; ++e) w[e] = digit_word<4>(m[e] * inv_q, t, over);
                store_digit_chunk<4>(F.D[0] + (size_t)r * digit_row_bytes(n, 4) + grp * 128 + hf * 16, w, top);
            } else {
#pragma unroll
                for (int e = 0; e < 16; ++e) { w[e] = digit_word<5>(m[e] * inv_q, t, over); top[e >> 2] |= t << (8 * (e & 3)); }
                store_digit_chunk<5>(F.D[0] + (size_t)r * digit_row_bytes(n, 5) + grp * 160 + hf * 16, w, top);
            }
        } else if (tier == TIER_F64) {
            double *d = F.F[0] + (size_t)r * F.ld64 + c0;
#pragma unroll
            for (int e = 0; e < 16; ++e) if (c0 + e < n) d[e] = m[e];
        }
        if (tier == TIER_PAIR || linear) {
#pragma unroll
            for (int e = 0; e < 16; ++e) w[e] = pair_word((float)(m[e] * (double)PAIR_SCALE_M));
            // a linear T reads M as pair planes in the X update, from the second iteration on: M_0 itself is needed by the chain only
            if (tier == TIER_PAIR) put_pair(F.P[0]);
        }
        if (linear) {
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float x = (float)((r == c0 + e ? (double)x1a : 0.0) - (double)x1e * m[e]);
                w[e] = c0 + e < n ? pair_word(x) : 0u;
                if (c0 + e <= r) F.Xout[(size_t)r * F.ldx + c0 + e] = x * inv_x;
            }
            put_pair(F.X[1]);
        }
    };
    const int si = (int)blockIdx.y >> 1, sj = (int)blockIdx.y & 1;
    if (ti == tj && si < sj) return;                             // covered by the mirrored sub-tile
    const int r0 = ti * 128 + si * 64, c0 = tj * 128 + sj * 64;
    if (r0 >= n || c0 >= n) return;
    {
        const int g = tid & 15, rw = tid >> 4;               // 16 groups of 4 columns x 16 rows
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            // P[rr][..] = A(r0 + rr, c0 ..), Q[rr][..] = A(c0 + rr, r0 ..)
            const int rr = rw + 16 * t;
            const int pr = r0 + rr, pc = c0 + 4 * g, qr = c0 + rr, qc = r0 + 4 * g;
            const float *ps = packed ? Ap + (size_t)(si * 64 + rr) * PACK_T + sj * 64 + 4 * g : F.A + (size_t)pr * lda + pc;
            if (vec && pr < n && pc + 4 <= n) {
                const float4 v = *reinterpret_cast<const float4 *>(ps);
                Pw[rr][4 * g] = v.x; Pw[rr][4 * g + 1] = v.y; Pw[rr][4 * g + 2] = v.z; Pw[rr][4 * g + 3] = v.w;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) Pw[rr][4 * g + e] = (pr < n && pc + e < n) ? ps[e] : 0.0f;
            }
            if (!packed) {
                const float *qs = F.A + (size_t)qr * lda + qc;
                if (vec && qr < n && qc + 4 <= n) {
                    const float4 v = *reinterpret_cast<const float4 *>(qs);
                    Qw[rr][4 * g] = v.x; Qw[rr][4 * g + 1] = v.y; Qw[rr][4 * g + 2] = v.z; Qw[rr][4 * g + 3] = v.w;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) Qw[rr][4 * g + e] = (qr < n && qc + e < n) ? qs[e] : 0.0f;
                }
            }
        }
    }
    __syncthreads();
    const int rr = tid >> 2, cg = (tid & 3) * 16;
    emit(r0 + rr, c0 + cg, [&](int e) {
        return packed ? (double)Pw[rr][cg + e] : 0.5 * ((double)Pw[rr][cg + e] + (double)Qw[cg + e][rr]);
    });
    if (!(ti == tj && si == sj))
        emit(c0 + rr, r0 + cg, [&](int e) {
            return packed ? (double)Pw[cg + e][rr] : 0.5 * ((double)Pw[cg + e][rr] + (double)Qw[rr][cg + e]);
        });
    if (over) F.flags[0] = 1;
}

// Planes from the matrices of a factor whose chain runs in fp64.  what 0: pair planes of E (the first iteration's
// becomes X_1), 1: of the next M, where the next iteration reads it so, 2: digits of M, where the chain goes over to them
// (into slot 1: E2 is dead, and slot 0 holds the fp64 M).
__global__ __launch_bounds__(256) void plane_from_f64_kernel(const FactorDev *fd, const FactorScal *fs, const int *state, int k, int what)
{
    const int f = blockIdx.y;
    const FactorScal &S = fs[f];
    if (what == 2 ? !S.from_f64 : S.tier != TIER_F64) return;
    const int st = state[f];
    if (st != ST_RUN && !(st == ST_LAST && what != 1)) return;
    if (what == 1 && !S.handover && !S.pair_m) return;
    const FactorDev &F = fd[f];
    const int n = F.n, per = plane_groups(n) * 2;
    const int id = blockIdx.x * 256 + threadIdx.x, r = id / per, c0 = (id % per) * 16;
    if (r >= n) return;
    const int slot = what == 0 ? 2 : 0;
    const double *src = F.F[slot] + (size_t)r * F.ld64 + c0;
    if (what == 2) {
        const double inv_q = ldexp(1.0, -S.dexp[0]);
        uint32_t wd[16], t;
        u32x4 top = {0u, 0u, 0u, 0u};
        bool over = false;
        const int grp = c0 >> 5, hf = (c0 >> 4) & 1;
        if (S.ns == 4) {
#pragma unroll
            for (int e = 0; e < 16; ++e) wd[e] = digit_word<4>((c0 + e < n ? src[e] : 0.0) * inv_q, t, over);
            store_digit_chunk<4>(F.D[1] + (size_t)r * digit_row_bytes(n, 4) + grp * 128 + hf * 16, wd, top);
        } else {
#pragma unroll
            for (int e = 0; e < 16; ++e) { wd[e] = digit_word<5>((c0 + e < n ? src[e] : 0.0) * inv_q, t, over); top[e >> 2] |= t << (8 * (e & 3)); }
            store_digit_chunk<5>(F.D[1] + (size_t)r * digit_row_bytes(n, 5) + grp * 160 + hf * 16, wd, top);
        }
        if (over) F.flags[0] = 1;
        return;
    }
    const bool x1 = what == 0 && k == 0;
    uint32_t w[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        double v = c0 + e < n ? src[e] : 0.0;
        if (x1) v = (r == c0 + e ? (double)S.x1a : 0.0) - (double)S.x1s * v;
        else v *= what == 0 ? (double)PAIR_SCALE_E : (double)PAIR_SCALE_M;
        w[e] = c0 + e < n ? pair_word((float)v) : 0u;
        if (x1 && c0 + e <= r) F.Xout[(size_t)r * F.ldx + c0 + e] = (float)(v / (double)S.x_scale);
    }
    char *d = (x1 ? F.X[1] : F.P[slot]) + (size_t)r * F.rowb + (c0 >> 5) * 128 + ((c0 >> 4) & 1) * 32;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        u32x4 hi, lo;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            hi[e] = __builtin_amdgcn_perm(w[8 * q + 2 * e + 1], w[8 * q + 2 * e], 0x05040100u);
            lo[e] = __builtin_amdgcn_perm(w[8 * q + 2 * e + 1], w[8 * q + 2 * e], 0x07060302u);
        }
        *(ASTERIA_GLOBAL u32x4 *)(d + q * 16) = hi;
        *(ASTERIA_GLOBAL u32x4 *)(d + 64 + q * 16) = lo;
    }
}

// Problem tables of the fp64 chain: E | E2 | W | M', one thread per factor.
struct PlaneF64Tables { GemmProblem *t[4]; };
__global__ void plane_f64_tables_kernel(const FactorDev *fd, FactorScal *fs, int cnt, int linear, PlaneF64Tables T)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= cnt) return;
    const FactorDev F = fd[i];
    const int ops[4] = {OP_SQ, OP_E2, OP_W, OP_M};
    GemmProblem p = {};
    p.M = p.N = p.K = F.n;
    p.state_idx = i; p.state_mask = 1 << ST_RUN;
    p.alpha = 1.0f; p.beta = 0.0f;
    p.lda = p.ldb = p.ldc = F.ld64;
    p.tile_start = F.tile_start;
    p.gate = &fs[i].tier;                            // TIER_F64 = 0
    p.partial = F.partial;
    for (int o = 0; o < 4; ++o) {
        const RootOperands r = root_operands(ops[o], linear != 0);
        GemmProblem q = p;
        q.A = F.F[r.A]; q.B = F.F[r.B]; q.C = F.F[r.C]; q.own = F.F[r.O1];
        q.coefd = &fs[i].prod[ops[o]].own1;
        q.flags = GEMM_SYM | (ops[o] == OP_M ? GEMM_EPI_RESID : 0);
        if (ops[o] == OP_SQ) q.state_mask |= 1 << ST_LAST;
        T.t[o][i] = q;
    }
}

// Outcome of every factor; the upper triangle of X where the last update did not complete the caller's matrix (a
// factor that ended with its first update, or ran out of iterations).  Grid: x = groups of rows, y = factor.
__global__ __launch_bounds__(256) void plane_finalize_kernel(const FactorDev *fd, const FactorScal *fs, const int *state, int first,
                                                             int32_t *info, int32_t *iters, float *resid, float *lambda_max)
{
    const int f = blockIdx.y;
    const FactorScal &S = fs[f];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (info) info[first + f] = S.info;
        if (iters) iters[first + f] = S.iters;
        if (resid) resid[first + f] = S.resid;
        if (lambda_max) lambda_max[first + f] = S.lam;
    }
    if (state[f] == ST_FAIL || S.xloc == 0) return;
    const FactorDev &F = fd[f];
    const int n = F.n;
    for (int r = blockIdx.x; r < n; r += gridDim.x)
        for (int c = threadIdx.x; c < r; c += 256) F.Xout[(size_t)c * F.ldx + r] = F.Xout[(size_t)r * F.ldx + c];
}

// ---- host --------------------------------------------------------------------------------------------
// Edge of the tiles of a pass's pair products.  Two workgroups of either the 64- or the 128-wide tiles fit a CU, so small ones pay
//   - where they are at most twice as many (n <= 64 and n in 129 .. 192): a large one is mostly empty;
//   - up to three of them per CU, and up to four where the large ones are more than one per CU.
// Roots in us at eps = 1e-6, 64 / 128-wide, by tiles of 128: n = 64 120 353 / 422, 400 616 / 687, 1000 1179 / 1352; n = 160 255 466 /
// 558, 501 744 / 784, 999 1314 / 1371; n = 200 and 333 in equal numbers 180 762 / 794, 252 839 / 814, 279 929 / 1007, 342 1053 / 1048, 396
// 1165 / 1116, 999 2405 / 2153; n = 512 200 859 / 884, 240 926 / 888, 280 1038 / 1130, 300 1149 / 1144, 400 1347 / 1269; n = 1024 180 1086 /
// 1141, 216 1197 / 1152, 252 1249 / 1179, 288 1526 / 1505.
// Large ones (one workgroup per CU) from two and a half rounds of the chip on, for matrices that their tiles cover no worse than
// 128-wide ones do.  128 over 256-wide, by tiles of 256: n = 768 558 0.96, 600 0.99, 650 1.00, 702 1.01, 750 1.04, 798 0.97, 852 1.00,
// 900 1.01, 1002 1.04; n = 900 560 0.97, 650 1.00, 700 1.01, 800 0.99, 850 0.99, 900 1.01, 1000 1.04; n = 1024 500 1.06, 560 0.99, 600
// 1.00, 650 1.01, 700 1.02, 750 1.06, 800 1.01, 900 1.04, 1000 1.06; n = 2048 396 1.01, 504 1.09, 612 1.06, 684 1.07, 900 1.05; n = 4096
// 408 1.06, 680 1.08; but n = 600 700 0.88, 1000 0.90 (a quarter more work), and n = 512 1800 0.96 (short K: the stores weigh more).
constexpr int PLANE_CUS = 256;
// Digit products in quarters of a tile up to as many halves.  Refresh in us, halves / quarters, by halves: 1 factor of n = 128 and one of 100 (4)
// 299.5 / 276.0, 512 and 400 (40) 441.5 / 412.7, 2 of 1024 (144) 682.9 / 656.1, 8 of 512 (160) 515.6 / 497.2, 120 of 128 (240) 446.8 / 430.8, 16 of 500 and
// 400 (320) 596 / 601, 240 of 128 and 100 (480) 644 / 657, 22 of 512 (440) 770 / 773.
constexpr int PLANE_QUARTERS = 256;
constexpr int PLANE_SMALL_TILES = 250, PLANE_LARGE_TILES = 700, PLANE_LARGE_N = 512;   // the first: of a factor that small tiles can serve
inline int pair_tile_edge(int tri64, int tri128, int tri256, int tri128_max, double work128, double work256, double n_mean)
{
    const bool small = tri64 <= 2 * tri128 || tri64 <= 768 || (tri128 > 256 && tri64 <= 1024);
    if (small && tri128_max < PLANE_SMALL_TILES) return 64;
    return tri256 >= PLANE_LARGE_TILES && work256 <= 1.03 * work128 && n_mean > (double)PLANE_LARGE_N ? 256 : 128;
}
// work of a factor's pair product in tiles of 128 x 128 x n: a diagonal tile of 256 takes three quarters of a whole one
inline double pair_work(int n, int tile)
{
    const double t = (n + tile - 1) / tile;
    return n * (tile == 256 ? 4.0 * (t * (t - 1) / 2 + 0.75 * t) : t * (t + 1) / 2);
}

inline size_t plane_pair_bytes(int n) { return Carver::need((size_t)n * pair_row_bytes(n), 1); }
// bytes of one chain slot: digits (5 at most), fp64 where that tier can occur
inline size_t plane_slot_bytes(int n, bool f64)
{
    size_t b = std::max(plane_pair_bytes(n), Carver::need((size_t)n * digit_row_bytes(n, 5), 1));
    if (f64) b = std::max(b, Carver::need((size_t)n * ((n + 1) & ~1), sizeof(double)));
    return b;
}
inline int plane_partials(int n)
{
    const int t = tri_tiles(n);
    return t < PLANE_SMALL_TILES ? std::max(2 * t, tri_tiles_of(n, 64)) : 2 * t;
}
// X_k, X_{k+1} and the chain slots.  The pair planes of M and E2 lie in slot 2, those of E and W in slot 3, over the
// digit or fp64 matrices of the prefix:
//   slot 2 (E, written by the first product of a T of degree 2): the pair planes of M are written by the last
//     product of an iteration, when E is dead, and read by one whose T is linear (no E) or that needs no prefix
//     matrices any more
//   slot 3 (W, written after the X update): the pair planes of E are read by the X update last, in every tier
inline size_t plane_factor_bytes(int n, bool prefix, bool f64)
{
    const size_t pair = plane_pair_bytes(n), slot = prefix ? plane_slot_bytes(n, f64) : pair;
    size_t b = 2 * pair + std::max(slot, 2 * pair) + slot + (prefix ? 2 * slot : 0);
    b += 2 * Carver::need(plane_partials(n), sizeof(float)) + 4 * sizeof(GemmProblem);
    const size_t t = tri_tiles(n);
    return b + (t + (size_t)tri_tiles_of(n, t < (size_t)PLANE_SMALL_TILES ? 64 : 256)) * sizeof(uint2);
}

}  // namespace asteria
