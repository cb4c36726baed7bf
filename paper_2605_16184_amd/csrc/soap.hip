// SOAP variant (paper Eq. 2):  N = Q_L phi(Q_L^T G Q_R) Q_R^T with phi = Adam in the rotated
// basis (asteria_soap_step), and the eigenbasis refresh Q <- qr(A Q).Q (asteria_soap_refresh).
//
// soap_step:   four grouped GEMMs (rotate in: G Q_R, then Q_L^T (.); rotate out: N' Q_R^T, then
//              Q_L (.)) around one HBM-streaming Adam kernel, on the bf16 matrix cores with every
//              fp32 operand split into two bf16 terms (16 bits kept, three MFMA passes per product,
//              two when G is bf16): a plain bf16 cast of an eigenbasis costs 0.1-0.5 relative error
//              in N, the split about 1e-5.  That kernel reads k-contiguous operands only, so the
//              call first writes Q_L^T and Q_R^T to the workspace, and the first product of each
//              rotation stores its result transposed.  Blocks whose shapes fill whole 256 x 256
//              tiles run the three split x split products on the 8-wavefront kernel of pgemm.h.
// soap_refresh: Z^T = Q^T A by one grouped GEMM (columns of Z become contiguous rows), then the
//              thin QR factor of Z with diag(R) > 0 - the same Q a Householder QR with that sign
//              convention returns, since the factorisation is unique - by block Gram-Schmidt
//              with re-orthogonalisation: panels of 128 columns; each panel is projected twice
//              against all finished panels (two grouped products on the fp16 matrix cores per
//              projection, so the O(n^3) work runs there), then orthonormalised by Cholesky QR
//              applied twice (soap_panel.h).  The second application removes the cond^2 * 2^-24
//              loss of the first, so ||Q^T Q - I|| ends at round-off level as long as
//              cond(Z) * 2^-24 < 1, and L's positive diagonal gives the diag(R) > 0 convention.
#include <algorithm>
#include <vector>

#include "common.h"
#include "gemm.h"
#include "gemm_bf16.h"
#include "pgemm.h"
#include "panel_product.h"
#include "soap_panel.h"

using namespace asteria;

namespace {

inline int ld4(int n) { return (n + 3) & ~3; }

// ---------------------------------------------------------------------------------------------
// Adam in the rotated basis, elementwise over every block.
struct AdamBlock {
    const float *Gr;   // rotated gradient G' (ld = ldw)
    float *M, *V;      // moments, in place
    float *Np;         // N' out (ld = ldw)
    int m, n, ldw, ldm, ldv;
    int row_start;     // first global row id of this block
};

__global__ __launch_bounds__(256) void adam_rotated_kernel(const AdamBlock *blocks, int nblocks,
                                                           float b1, float b2, float eps,
                                                           float inv_c1, float inv_c2)
{
    // one workgroup per matrix row
    int lo = 0, hi = nblocks - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (blocks[mid].row_start <= (int)blockIdx.x) lo = mid; else hi = mid - 1;
    }
    const AdamBlock &B = blocks[lo];
    const int row = (int)blockIdx.x - B.row_start;
    const float *__restrict__ g = B.Gr + (size_t)row * B.ldw;
    float *__restrict__ mm = B.M + (size_t)row * B.ldm;
    float *__restrict__ vv = B.V + (size_t)row * B.ldv;
    float *__restrict__ np = B.Np + (size_t)row * B.ldw;
    for (int j = threadIdx.x; j < B.n; j += 256) {
        const float gj = g[j];
        const float m1 = b1 * mm[j] + (1.0f - b1) * gj;
        const float v1 = b2 * vv[j] + (1.0f - b2) * gj * gj;
        mm[j] = m1;
        vv[j] = v1;
        np[j] = (m1 * inv_c1) / (sqrtf(v1 * inv_c2) + eps);
    }
}

// ---------------------------------------------------------------------------------------------
// dst = src^T for a batch of fp32 matrices, 32 x 32 tiles through LDS (reads and writes along rows)
struct TransposeF32Job {
    const float *src;   // rows x cols, ld = lds_
    float *dst;         // cols x rows, ld = ldd
    int rows, cols, lds_, ldd;
    int tile_start;
    int pad_;
};

__global__ __launch_bounds__(256) void transpose_f32_kernel(const TransposeF32Job *jobs, int njobs)
{
    int lo = 0, hi = njobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (jobs[mid].tile_start <= (int)blockIdx.x) lo = mid; else hi = mid - 1;
    }
    const TransposeF32Job &J = jobs[lo];
    const int lt = (int)blockIdx.x - J.tile_start;
    const int tcols = (J.cols + 31) / 32;
    const int ti = lt / tcols, tj = lt % tcols;
    __shared__ float tile[32][33];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int rr = ty; rr < 32; rr += 8) {
        const int r = ti * 32 + rr, c = tj * 32 + tx;
        tile[rr][tx] = (r < J.rows && c < J.cols) ? J.src[(size_t)r * J.lds_ + c] : 0.0f;
    }
    __syncthreads();
    for (int rr = ty; rr < 32; rr += 8) {
        const int r = tj * 32 + rr, c = ti * 32 + tx;   // element (r, c) of dst = src(c, r)
        if (r < J.cols && c < J.rows) J.dst[(size_t)r * J.ldd + c] = tile[tx][rr];
    }
}

// ---------------------------------------------------------------------------------------------
// Eigenbasis refresh (panel steps: soap_panel.h)
// Panels whose rows are projected together in the first sweep: what is finished before the first of them is read once for
// all, what is finished since, once for each.  Refresh of the 1.1B model: 1 panel 128.3 ms, 2: 123.1, 3: 123.8, 4: 123.4
// (two streams; the coefficients of each take 128 n floats).
constexpr int QR_AHEAD = 2;
constexpr int QR_STATE_STRIDE = (int)(sizeof(QrFactor) / sizeof(int));
static_assert(sizeof(QrFactor) % sizeof(int) == 0, "state words are addressed as ints inside the factor array");

// a_scale = p_scale = largest power of two with 2^e tr|A| <= 30000 (|Z_ij| <= ||A||_2 <= tr A for a
// positive semi-definite A and orthonormal Q); one wavefront per factor
__global__ __launch_bounds__(64) void qr_scale_kernel(QrFactor *fs, int nf)
{
    const int f = blockIdx.x;
    if (f >= nf) return;
    const float *a = fs[f].A;
    const int n = fs[f].n, ld = fs[f].lda;
    double t = 0.0;
    for (int i = threadIdx.x; i < n; i += 64) t += fabs((double)a[(size_t)i * ld + i]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
    if (threadIdx.x == 0) {
        int e = (t > 0.0 && t < 1e300) ? (int)floor(log2(30000.0 / t)) : 0;
        e = e < -100 ? -100 : (e > 100 ? 100 : e);
        const float sc = (float)ldexp(1.0, e);
        fs[f].a_scale = sc;
        fs[f].p_scale = sc;
    }
}

constexpr int QR_MAXN = 1 << 20;

__global__ void qr_info_kernel(const QrFactor *fs, int nf, int32_t *info)
{
    const int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f < nf && info) info[fs[f].out_index] = fs[f].bad ? ASTERIA_INFO_NOT_PD : ASTERIA_INFO_OK;
}

// Q <- Q^T in place: pairs of mirrored 32 x 32 tiles swapped through LDS.  Grid: x = tile (row-major
// over the largest factor's tile grid; tiles below the diagonal or outside this factor do nothing),
// y = factor.
__global__ __launch_bounds__(256) void transpose_inplace_kernel(const QrFactor *fs)
{
    const QrFactor &F = fs[blockIdx.y];
    if (F.Qt != F.Qout) return;                       // the caller keeps Q^T beside Q: nothing to transpose
    const int tpr = (F.n + 31) / 32, tmax = (int)rintf(sqrtf((float)gridDim.x));
    const int ti = (int)blockIdx.x / tmax, tj = (int)blockIdx.x % tmax;
    if (ti > tj || tj >= tpr) return;
    __shared__ float up[32][33], lo[32][33];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int r = ty; r < 32; r += 8) {
        const int i = ti * 32 + r, c = tj * 32 + tx;     // upper tile (ti, tj)
        up[r][tx] = (i < F.n && c < F.n) ? F.Qout[(size_t)i * F.ldq + c] : 0.0f;
        const int i2 = tj * 32 + r, c2 = ti * 32 + tx;   // its mirror (tj, ti)
        lo[r][tx] = (i2 < F.n && c2 < F.n) ? F.Qout[(size_t)i2 * F.ldq + c2] : 0.0f;
    }
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
        const int i = ti * 32 + r, c = tj * 32 + tx;
        if (i < F.n && c < F.n) F.Qout[(size_t)i * F.ldq + c] = lo[tx][r];
        const int i2 = tj * 32 + r, c2 = ti * 32 + tx;
        if (ti != tj && i2 < F.n && c2 < F.n) F.Qout[(size_t)i2 * F.ldq + c2] = up[tx][r];
    }
}

// Q = I for every factor of the group (the refresh then starts from the identity)
__global__ __launch_bounds__(256) void set_identity_kernel(const QrFactor *fs)
{
    const QrFactor &F = fs[blockIdx.y];
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < (size_t)F.n * F.n; e += (size_t)gridDim.x * 256) {
        const int i = (int)(e / F.n), j = (int)(e % F.n);
        F.Qout[(size_t)i * F.ldq + j] = (i == j) ? 1.0f : 0.0f;
        if (F.Qt != F.Qout) F.Qt[(size_t)i * F.ldqt + j] = (i == j) ? 1.0f : 0.0f;
    }
}

// Qt <- Q^T where the caller keeps Q^T beside Q and the buffer does not hold it yet: 32 x 32 tiles through LDS.
// Grid: x = tile of the largest factor's tile grid, y = factor; factors without such a buffer do nothing.
__global__ __launch_bounds__(256) void keep_qt_kernel(const QrFactor *fs)
{
    const QrFactor &F = fs[blockIdx.y];
    if (F.Qt == F.Qout) return;
    const int tpr = (F.n + 31) / 32, tmax = (int)rintf(sqrtf((float)gridDim.x));
    const int ti = (int)blockIdx.x / tmax, tj = (int)blockIdx.x % tmax;
    if (ti >= tpr || tj >= tpr) return;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    __shared__ float tile[32][33];
    for (int r = ty; r < 32; r += 8) {
        const int i = ti * 32 + r, c = tj * 32 + tx;
        tile[r][tx] = (i < F.n && c < F.n) ? F.Qout[(size_t)i * F.ldq + c] : 0.0f;
    }
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
        const int i = tj * 32 + r, c = ti * 32 + tx;     // Qt(i, c) = Q(c, i)
        if (i < F.n && c < F.n) F.Qt[(size_t)i * F.ldqt + c] = tile[tx][r];
    }
}

// Column order of the basis before the refresh (the order SOAP uses): est_i = q_i^T A q_i, largest
// first, ties by index.  With Q^T in the caller's buffer (rows q_i^T) and Z^T = Q^T A already formed,
// est_i is the dot product of row i of the two; one wavefront per row, fp64 sums.
__global__ __launch_bounds__(256) void sort_estimate_kernel(const QrFactor *fs)
{
    const QrFactor &F = fs[blockIdx.y];
    const int row = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (row >= F.n) return;
    const float *q = F.Qt + (size_t)row * F.ldqt, *z = F.Zt + (size_t)row * F.ldz;
    double s = 0.0;
    for (int k = lane; k < F.n; k += 64) s += (double)q[k] * (double)z[k];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    // the order has to be total, or ranks collide and entries of perm stay unwritten: not a number comes last
    if (lane == 0) F.est[row] = s == s ? s : -INFINITY;
}

// rank of every estimate: the number of columns that come before it (larger estimate, or equal and a
// lower index); perm[rank] = column.
// Sixteen lanes share a column: with one each, n serial comparisons (74 us at n = 1024) were as long as a panel's Gram
// matrix, Cholesky factor and inverse.
constexpr int RANK_LANES = 16, RANK_COLS = 256 / RANK_LANES;
__global__ __launch_bounds__(256) void sort_rank_kernel(const QrFactor *fs)
{
    const QrFactor &F = fs[blockIdx.y];
    const int n = F.n, i = (int)blockIdx.x * RANK_COLS + (int)threadIdx.x / RANK_LANES, l = (int)threadIdx.x % RANK_LANES;
    if ((int)blockIdx.x * RANK_COLS >= n) return;
    const ASTERIA_GLOBAL double *est = (const ASTERIA_GLOBAL double *)F.est;
    const double mine = est[min(i, n - 1)];
    int rank = 0;
#pragma unroll 4
    for (int j = l; j < n; j += RANK_LANES) {
        const double o = est[j];
        rank += (o > mine || (o == mine && j < i)) ? 1 : 0;
    }
#pragma unroll
    for (int off = RANK_LANES / 2; off > 0; off >>= 1) rank += __shfl_xor(rank, off, 64);
    if (l == 0 && i < n) {
        F.perm[rank] = i;
        if (F.perm_out) F.perm_out[rank] = i;
    }
}

// rows of Z^T gathered in the new order, through the caller's Q buffer (free between the product that
// formed Z^T and the first finished panel): phase 0: Q[r] = Zt[perm[r]]; phase 1: Zt[r] = Q[r]
__global__ __launch_bounds__(256) void sort_gather_kernel(const QrFactor *fs, int phase)
{
    const QrFactor &F = fs[blockIdx.y];
    const int row = (int)blockIdx.x;
    if (row >= F.n) return;
    const float *src = phase == 0 ? F.Zt + (size_t)F.perm[row] * F.ldz : F.Qout + (size_t)row * F.ldq;
    float *dst = phase == 0 ? F.Qout + (size_t)row * F.ldq : F.Zt + (size_t)row * F.ldz;
    for (int k = threadIdx.x; k < F.n; k += 256) dst[k] = src[k];
}

// Products of fp32 matrices over two fp16 terms each, in one launch: `tiles` small tiles of whole-tile problems, and the tiles of
// gemm_bf16.h of those with a remainder in `ragged`.  (4 ragged tiles of n = 76 in a launch of their own: 23 us on top of the 59
// of 456 whole ones.)
__global__ __launch_bounds__(2 * PG_SMALL_TILE, 2) void product_f16_kernel(const PlaneProblem *__restrict__ probs, int nprobs, int tiles,
                                                                           const GemmProblem *__restrict__ ragged, int nragged, int ragged_tiles)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    bool second;
    const int t = joint_tile(ragged_tiles, tiles, second);
    if (t < 0) return;
    if (second) pgemm_tile<2, true, PG_SMALL_TILE>(probs, nprobs, t, smem_raw);
    else gemm_bf16_tile<float, float, 2, 2, true>(ragged, nragged, t, nullptr, smem_raw);
}

hipError_t launch_product_f16(const PlaneProblem *probs, int nprobs, int tiles, const GemmProblem *ragged, int nragged,
                              int ragged_tiles, hipStream_t stream)
{
    if (tiles + ragged_tiles <= 0) return hipSuccess;
    constexpr size_t lds = pg_lds_bytes(2, PG_SMALL_TILE);
    static_assert(lds >= gemm_bf16_lds<float, float, 2, 2>(), "either kind of tile");
    static bool configured[MAX_DEVICES] = {};
    if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(product_f16_kernel), lds, configured); e != hipSuccess) return e;
    profile_begin(tiles > 0 ? 513 : 224, stream);
    hipLaunchKernelGGL(product_f16_kernel, dim3(joint_grid(ragged_tiles, tiles)), dim3(2 * PG_SMALL_TILE), lds, stream, probs, nprobs, tiles, ragged, nragged,
                       ragged_tiles);
    profile_end(stream);
    return hipGetLastError();
}

// Problem tables of one group of factors, written on the device from the factor descriptors (as host
// tables they travel as kernel arguments: about 500 upload launches per group of the 1B-model workload).
// The factors of a group are sorted by size, largest first, so those that have panel j are the first
// count_j of the group and the entry of factor i in any table of panel j is entry i of that panel's run.
struct RefreshTables {
    GemmProblem *z;                    // Z^T = Q^T A of the factors that are no whole tiles
    PlaneProblem *zp;                  // the same of those that are, the first zp_large on large tiles
    int zp_large;
    // projection coefficients, projection: a factor has an entry in both kinds of table, with no tiles in the one that it
    // does not use (whole-panel factors: p1, p2)
    GemmProblem *t1, *t2;
    PanelProblem *f1, *f2;             // whole-panel factors, first sweep
    PanelProblem *p1, *p2;             // the later ones
    const int *off;                    // np + 1: start of panel j's run in the tables t1 .. p2
    const int *whole;                  // cnt + 1: whole-panel factors before i
    const int *pt;                     // cnt + 1: tile columns (ceil(n / 128)) of the other factors before i
    const int *pp[2];                  // cnt + 1: tiles of 128, of 256 columns of the whole-panel factors before i
    const int *pz;                     // cnt: first tile of factor i in the launch of its Z product
    const int *slot;                   // cnt: its entry there, s in z or -1 - s in zp
    int share;                         // see refresh_shares
};

__global__ __launch_bounds__(128) void refresh_tables_kernel(QrFactor *fs, int cnt, RefreshTables T)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x, j = blockIdx.y;
    if (i >= cnt) return;
    const QrFactor F = fs[i];
    const float *a_scale = &fs[i].a_scale, *p_scale = &fs[i].p_scale;
    const int tn = (F.n + BN - 1) / BN;
    GemmProblem p = {};
    p.alpha = 1.0f; p.beta = 0.0f;
    if (j == 0) {
        // Z^T = Q^T A on the fp16 cores (two terms per operand): A'(i, k) = Q^T[i][k] - the caller's Q has
        // been transposed in place by then, or the caller keeps Q^T -, scaled by 2^14, and B'(j, k) = A[j][k] (A is symmetric),
        // scaled by the factor's a_scale; both k-contiguous
        const int slot = T.slot[i];
        if (slot < 0) {
            PlaneProblem g = {};
            g.M = g.N = g.K = F.n; g.tiles_n = F.n / (-1 - slot < T.zp_large ? PG_TILE : PG_SMALL_TILE);
            g.A = F.Qt; g.lda = F.ldqt; g.B = F.A; g.ldb = F.lda; g.C32 = F.Zt; g.ldc32 = F.ldz;
            g.sa = QR_UNIT_SCALE; g.sb_dev = a_scale;
            g.tile_start = T.pz[i];
            T.zp[-1 - slot] = g;
        } else {
            GemmProblem g = p;
            g.state_idx = -1; g.state_mask = ~0;
            g.M = g.N = g.K = F.n; g.tiles_n = tn;
            g.A = F.Qt; g.lda = F.ldqt; g.B = F.A; g.ldb = F.lda; g.C = F.Zt; g.ldc = F.ldz;
            g.sa = QR_UNIT_SCALE; g.sb_dev = a_scale;
            g.tile_start = T.pz[i];
            T.z[slot] = g;
        }
    }
    if (F.n <= j * QR_PANEL) return;
    const int e = T.off[j] + i;
    const int rows = min(QR_PANEL, F.n - j * QR_PANEL), done = j * QR_PANEL;
    float *Pt = F.Zt + (size_t)done * F.ldz;
    if (j == 0) return;
    // runs while the factor's state word (`run`, or `skip3` in the third sweep) is 0
    p.state_idx = i * QR_STATE_STRIDE; p.state_mask = 1;
    // C = P Q_done^T: rows of the panel against the finished rows, contraction over n; on the fp16 cores
    // the panel rows are scaled by the factor's p_scale, the finished rows are orthonormal
    p.M = rows; p.N = done; p.K = F.n; p.tiles_n = j;
    p.A = Pt; p.lda = F.ldz; p.B = F.Zt; p.ldb = F.ldz; p.C = F.cbuf; p.ldc = F.ldz;
    p.tile_start = (i - T.whole[i]) * j;       // every factor of the run has j tile columns here
    p.sa_dev = p_scale; p.sb = QR_UNIT_SCALE;
    T.t1[e] = p;
    // whole panels.  First sweep: QR_AHEAD panels at a time against what is finished before the first of them, and each
    // of the others against those since then, `near` rows of it
    const int near = (j % QR_AHEAD) * QR_PANEL, ahead = min(QR_AHEAD, (int)gridDim.y - j);
    PanelProblem w = {};
    w.ldx = F.ldz; w.Y = Pt; w.ldy = F.ldz; w.C = F.cbuf; w.ldc = F.ldz; w.K = F.n;
    w.x_scale = QR_UNIT_SCALE; w.y_scale = p_scale; w.state_idx = i * QR_STATE_STRIDE;
    w.X = F.Zt; w.N = done; w.panels = w.slots = 1;
    w.start[0] = T.whole[i] * j; w.start[1] = T.whole[i] * ((j + 1) / 2);
    T.p1[e] = w;
    PanelProblem w2 = w;
    w2.X = F.Qout; w2.ldx = F.ldq; w2.Y = F.cbuf; w2.C = Pt; w2.N = F.n; w2.K = done;
    w2.subtract = 1;
    w2.start[0] = T.pp[0][i]; w2.start[1] = T.pp[1][i];
    T.p2[e] = w2;
    if (near > 0) {
        if (!T.share && done > near) {
            // no panel takes part in another's pass: this one's own part of it, in the entry that the panel before leaves free
            static_assert(QR_AHEAD == 2, "one free entry per far part");
            const int far = j - 1, e0 = T.off[far] + i;
            PanelProblem v = w, v2 = w2;
            v.N = v2.K = done - near;
            v.start[0] = T.whole[i] * far; v.start[1] = T.whole[i] * ((far + 1) / 2);
            T.f1[e0] = v;
            T.f2[e0] = v2;
        }
        w.X = F.Zt + (size_t)(done - near) * F.ldz; w.N = near;
        w.start[0] = T.whole[i] * (near / QR_PANEL); w.start[1] = T.whole[i] * ((near / QR_PANEL + 1) / 2);
        w2.X = F.Qout + (done - near); w2.K = near;
    } else if (T.share) {
        w.slots = w2.slots = ahead;
        w.panels = w2.panels = min(ahead, F.n / QR_PANEL - j);
        w.start[0] *= ahead; w.start[1] *= ahead; w2.start[0] *= ahead; w2.start[1] *= ahead;
    }
    if (near > 0 || T.share) {
        T.f1[e] = w;
        T.f2[e] = w2;
    }
    // P <- P - C Q_done: contraction over the finished rows, which the caller's Q already holds as
    // columns (k contiguous); the coefficients share the scale of the panel rows
    p.alpha = -1.0f; p.beta = 1.0f;
    p.M = rows; p.N = F.n; p.K = done; p.tiles_n = tn;
    p.A = F.cbuf; p.lda = F.ldz; p.B = F.Qout; p.ldb = F.ldq; p.C = Pt; p.ldc = F.ldz;
    p.tile_start = T.pt[i];
    T.t2[e] = p;
}

asteria_status validate_step(const asteria_sblock *b, int nblocks, float b1, float b2, float eps, int t)
{
    if (!b || nblocks <= 0 || t < 1) return ASTERIA_INVALID_ARG;
    if (!(b1 >= 0.0f && b1 < 1.0f) || !(b2 >= 0.0f && b2 < 1.0f) || !(eps >= 0.0f)) return ASTERIA_INVALID_ARG;
    for (int i = 0; i < nblocks; ++i) {
        const asteria_sblock &k = b[i];
        if (!k.G || (!k.QL && !k.QR) || !k.M || !k.V || !k.N) return ASTERIA_INVALID_ARG;   // one side may be the identity
        if (k.m <= 0 || k.n <= 0) return ASTERIA_INVALID_ARG;
        if (k.ldg < k.n || (k.QL && k.ldql < k.m) || (k.QR && k.ldqr < k.n) || k.ldm < k.n || k.ldv < k.n || k.ldn < k.n)
            return ASTERIA_INVALID_ARG;
        if (!valid_dtype(k.g_dtype)) return ASTERIA_INVALID_ARG;
        if ((k.QLt && k.ldqlt < k.m) || (k.QRt && k.ldqrt < k.n)) return ASTERIA_INVALID_ARG;
    }
    return ASTERIA_OK;
}

// The same transposition for descriptors that travel as kernel arguments (asteria_transpose has no workspace).
constexpr int TRANSPOSE_CHUNK = 64;
struct TransposeChunk {
    TransposeF32Job job[TRANSPOSE_CHUNK];
};

__global__ __launch_bounds__(256) void transpose_chunk_kernel(TransposeChunk c, int njobs)
{
    int lo = 0, hi = njobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (c.job[mid].tile_start <= (int)blockIdx.x) lo = mid; else hi = mid - 1;
    }
    const TransposeF32Job &J = c.job[lo];
    const int lt = (int)blockIdx.x - J.tile_start;
    const int tcols = (J.cols + 31) / 32;
    const int ti = lt / tcols, tj = lt % tcols;
    __shared__ float tile[32][33];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int rr = ty; rr < 32; rr += 8) {
        const int r = ti * 32 + rr, cc = tj * 32 + tx;
        tile[rr][tx] = (r < J.rows && cc < J.cols) ? J.src[(size_t)r * J.lds_ + cc] : 0.0f;
    }
    __syncthreads();
    for (int rr = ty; rr < 32; rr += 8) {
        const int r = tj * 32 + rr, cc = ti * 32 + tx;   // element (r, cc) of dst = src(cc, r)
        if (r < J.cols && cc < J.rows) J.dst[(size_t)r * J.ldd + cc] = tile[tx][rr];
    }
}

}  // namespace

extern "C" asteria_status asteria_transpose(const asteria_tpair *items, int nitems, void *stream_)
{
    if (!items || nitems <= 0) return ASTERIA_INVALID_ARG;
    for (int i = 0; i < nitems; ++i) {
        const asteria_tpair &t = items[i];
        if (!t.src || !t.dst || t.rows <= 0 || t.cols <= 0 || t.lds < t.cols || t.ldd < t.rows) return ASTERIA_INVALID_ARG;
    }
    hipStream_t stream = reinterpret_cast<hipStream_t>(stream_);
    for (int first = 0; first < nitems; first += TRANSPOSE_CHUNK) {
        const int cnt = std::min(TRANSPOSE_CHUNK, nitems - first);
        TransposeChunk c;
        memset(&c, 0, sizeof(c));
        int tiles = 0;
        for (int i = 0; i < cnt; ++i) {
            const asteria_tpair &t = items[first + i];
            TransposeF32Job &J = c.job[i];
            J.src = t.src; J.dst = t.dst; J.rows = t.rows; J.cols = t.cols; J.lds_ = t.lds; J.ldd = t.ldd;
            J.tile_start = tiles;
            tiles += ((t.rows + 31) / 32) * ((t.cols + 31) / 32);
        }
        hipLaunchKernelGGL(transpose_chunk_kernel, dim3(tiles), dim3(256), 0, stream, c, cnt);
        ASTERIA_HIP_TRY(hipGetLastError());
    }
    return ASTERIA_OK;
}

extern "C" size_t asteria_soap_step_workspace_bytes(const asteria_sblock *blocks, int nblocks)
{
    if (!blocks || nblocks <= 0) return 0;
    size_t bytes = 4 * Carver::need((size_t)nblocks, sizeof(GemmProblem)) + Carver::need((size_t)nblocks, sizeof(AdamBlock)) +
                   Carver::need(2 * (size_t)nblocks, sizeof(TransposeF32Job)) +
                   3 * Carver::need((size_t)nblocks, sizeof(PlaneProblem)) + Carver::need(4 * (size_t)nblocks, sizeof(GemmProblem)) + 2048;
    for (int i = 0; i < nblocks; ++i) {
        const int m = blocks[i].m, n = blocks[i].n;
        bytes += 2 * Carver::need((size_t)m * ld4(n), sizeof(float));      // G' / N' (m x n)
        bytes += Carver::need((size_t)n * ld4(m), sizeof(float));          // transposed intermediate (n x m)
        if (!blocks[i].QLt) bytes += Carver::need((size_t)m * ld4(m), sizeof(float));   // Q_L^T, unless the caller keeps it
        if (!blocks[i].QRt) bytes += Carver::need((size_t)n * ld4(n), sizeof(float));   // Q_R^T
    }
    return bytes;
}

extern "C" asteria_status asteria_soap_step(const asteria_sblock *blocks, int nblocks,
                                            float beta1, float beta2, float adam_eps, int step_t,
                                            void *ws, size_t ws_bytes, void *stream_)
{
    asteria_status st = validate_step(blocks, nblocks, beta1, beta2, adam_eps, step_t);
    if (st != ASTERIA_OK) return st;
    if (!ws || ws_bytes < asteria_soap_step_workspace_bytes(blocks, nblocks)) return ASTERIA_WORKSPACE_TOO_SMALL;
    if (reinterpret_cast<uintptr_t>(ws) & 255u) return ASTERIA_INVALID_ARG;   // workspace must be 256-byte aligned
    hipStream_t stream = reinterpret_cast<hipStream_t>(stream_);

    Carver cv(ws);
    GemmProblem *d_g[4];
    for (int i = 0; i < 4; ++i) d_g[i] = cv.take<GemmProblem>(nblocks);
    AdamBlock *d_ab = cv.take<AdamBlock>(nblocks);
    TransposeF32Job *d_tj = cv.take<TransposeF32Job>(2 * (size_t)nblocks);
    PlaneProblem *d_f[3];
    for (int i = 0; i < 3; ++i) d_f[i] = cv.take<PlaneProblem>(nblocks);
    std::vector<PlaneProblem> f1, f2, f3, f4;   // products of blocks that fill whole 256 x 256 tiles (the first one: bf16 gradients)
    int tilesf = 0;
    std::vector<GemmProblem> g1[2], g2, g3, g4;
    // one-sided blocks (Q_L or Q_R absent = the identity on that side, e.g. a dimension above the
    // preconditioner cap): one product per rotation, on the fp32 matrix cores, operands read in place
    std::vector<GemmProblem> oL1[2], oL2, oR1[2], oR2;     // left only: Q_L^T G, Q_L N';  right only: G Q_R, N' Q_R^T
    int tL1[2] = {0, 0}, tL2 = 0, tR1[2] = {0, 0}, tR2 = 0;
    std::vector<AdamBlock> ab;
    std::vector<TransposeF32Job> tj;
    int tiles1[2] = {0, 0}, tiles1f = 0, tiles = 0, tilesT = 0, rows = 0, ttiles = 0;
    // 256 x 256 tiles the call offers to the kernels of pgemm.h, and their sum of K (transposes made here lie aligned in the workspace)
    long long t1 = 0, tk1 = 0, t2 = 0, tk2 = 0;
    auto whole1 = [](const asteria_sblock &k) {
        return k.QL && k.QR && k.g_dtype == ASTERIA_BF16 && pg_bf16_operand_ok(k.G, k.m, k.n, k.ldg) &&
               (k.n % PG_TILE) == 0 && (!k.QRt || pg_f32_operand_ok(k.QRt, k.n, k.n, k.ldqrt));
    };
    for (int i = 0; i < nblocks; ++i) {
        const asteria_sblock &k = blocks[i];
        if (!k.QL || !k.QR || k.m % PG_TILE || k.n % PG_TILE) continue;
        const long long t = (long long)(k.m / PG_TILE) * (k.n / PG_TILE);
        if (whole1(k)) { t1 += t; tk1 += t * k.n; }
        t2 += t; tk2 += t * (k.m + k.n) / 2;
    }
    const bool use1 = pg_take_large_tiles(t1, tk1), use2 = pg_take_large_tiles(t2, tk2);
    for (int i = 0; i < nblocks; ++i) {
        const asteria_sblock &k = blocks[i];
        const int ldw = ld4(k.n), ldt = ld4(k.m);
        const int ldqlt = k.QLt ? k.ldqlt : ld4(k.m), ldqrt = k.QRt ? k.ldqrt : ld4(k.n);
        float *Gr = cv.take<float>((size_t)k.m * ldw);   // G' (m x n)
        float *Np = cv.take<float>((size_t)k.m * ldw);   // N' (m x n)
        if (!k.QL || !k.QR) {
            const int tm1 = (k.m + BM - 1) / BM, tn1 = (k.n + BN - 1) / BN;
            GemmProblem p;
            memset(&p, 0, sizeof(p));
            p.state_idx = -1; p.state_mask = ~0; p.alpha = 1.0f; p.beta = 0.0f;
            p.M = k.m; p.N = k.n; p.tiles_n = tn1;
            if (k.QL) {
                // G' = Q_L^T G: A'(i, l) = Q_L[l][i], B'(j, l) = G[l][j], both k-major
                p.K = k.m; p.A = k.QL; p.lda = k.ldql; p.B = k.G; p.ldb = k.ldg; p.C = Gr; p.ldc = ldw;
                p.tile_start = tL1[k.g_dtype]; tL1[k.g_dtype] += tm1 * tn1;
                oL1[k.g_dtype].push_back(p);
                // N = Q_L N': A'(i, l) = Q_L[i][l], B'(j, l) = N'[l][j] (k-major)
                p.A = k.QL; p.lda = k.ldql; p.B = Np; p.ldb = ldw; p.C = k.N; p.ldc = k.ldn;
                p.tile_start = tL2; tL2 += tm1 * tn1;
                oL2.push_back(p);
            } else {
                // G' = G Q_R: A' = G, B'(j, l) = Q_R[l][j] (k-major)
                p.K = k.n; p.A = k.G; p.lda = k.ldg; p.B = k.QR; p.ldb = k.ldqr; p.C = Gr; p.ldc = ldw;
                p.tile_start = tR1[k.g_dtype]; tR1[k.g_dtype] += tm1 * tn1;
                oR1[k.g_dtype].push_back(p);
                // N = N' Q_R^T: A' = N', B'(j, l) = Q_R[j][l]
                p.A = Np; p.lda = ldw; p.B = k.QR; p.ldb = k.ldqr; p.C = k.N; p.ldc = k.ldn;
                p.tile_start = tR2; tR2 += tm1 * tn1;
                oR2.push_back(p);
            }
            AdamBlock a1;
            a1.Gr = Gr; a1.M = k.M; a1.V = k.V; a1.Np = Np; a1.m = k.m; a1.n = k.n; a1.ldw = ldw; a1.ldm = k.ldm; a1.ldv = k.ldv;
            a1.row_start = rows; rows += k.m;
            ab.push_back(a1);
            continue;
        }
        float *Tt = cv.take<float>((size_t)k.n * ldt);   // (G Q_R)^T, later (N' Q_R^T)^T  (n x m)
        // transposed bases: the caller's copies, or made here
        const float *QLt = k.QLt, *QRt = k.QRt;
        TransposeF32Job t;
        memset(&t, 0, sizeof(t));
        if (!QLt) {
            float *dst = cv.take<float>((size_t)k.m * ldqlt);
            t.src = k.QL; t.dst = dst; t.rows = k.m; t.cols = k.m; t.lds_ = k.ldql; t.ldd = ldqlt;
            t.tile_start = ttiles; ttiles += ((k.m + 31) / 32) * ((k.m + 31) / 32);
            tj.push_back(t);
            QLt = dst;
        }
        if (!QRt) {
            float *dst = cv.take<float>((size_t)k.n * ldqrt);
            t.src = k.QR; t.dst = dst; t.rows = k.n; t.cols = k.n; t.lds_ = k.ldqr; t.ldd = ldqrt;
            t.tile_start = ttiles; ttiles += ((k.n + 31) / 32) * ((k.n + 31) / 32);
            tj.push_back(t);
            QRt = dst;
        }
        const int tm = (k.m + BM - 1) / BM, tn = (k.n + BN - 1) / BN;
        GemmProblem p;
        memset(&p, 0, sizeof(p));
        p.state_idx = -1; p.state_mask = ~0; p.alpha = 1.0f; p.beta = 0.0f;
        // 1: (G Q_R)^T:   A' = G (m x n), B' = Q_R^T (B'(j, k) = Q_R[k][j]); m x n result stored transposed
        // (whole-tile blocks with bf16 gradients: (G Q_R)^T = Q_R^T G^T, A' = Q_R^T, B' = G)
        p.M = k.m; p.N = k.n; p.K = k.n; p.tiles_n = tn;
        if (use1 && whole1(k)) {
            PlaneProblem q;
            memset(&q, 0, sizeof(q));
            q.A = QRt; q.lda = ldqrt; q.B = k.G; q.ldb = k.ldg; q.C32 = Tt; q.ldc32 = ldt;
            q.M = k.n; q.N = k.m; q.K = k.n; q.tiles_n = k.m / PG_TILE;
            q.tile_start = tiles1f; tiles1f += (k.n / PG_TILE) * q.tiles_n;
            f1.push_back(q);
        } else {
            p.A = k.G; p.lda = k.ldg; p.B = QRt; p.ldb = ldqrt; p.C = Tt; p.ldc = ldt; p.flags = GEMM_STORE_T;
            p.tile_start = tiles1[k.g_dtype]; tiles1[k.g_dtype] += tm * tn;
            g1[k.g_dtype].push_back(p);
        }
        const bool fast = use2 && pg_f32_operand_ok(QLt, k.m, k.m, ldqlt) && pg_f32_operand_ok(Tt, k.n, k.m, ldt) &&
                          pg_f32_operand_ok(Np, k.m, k.n, ldw) && pg_f32_operand_ok(k.QR, k.n, k.n, k.ldqr) &&
                          pg_f32_operand_ok(k.QL, k.m, k.m, k.ldql);
        if (fast) {
            PlaneProblem q;
            memset(&q, 0, sizeof(q));
            q.M = k.m; q.N = k.n; q.tiles_n = k.n / PG_TILE; q.tile_start = tilesf;
            q.K = k.m; q.A = QLt; q.lda = ldqlt; q.B = Tt; q.ldb = ldt; q.C32 = Gr; q.ldc32 = ldw; q.flags = 0;
            f2.push_back(q);
            PlaneProblem q3 = q;                      // (N' Q_R^T)^T = Q_R N'^T
            q3.M = k.n; q3.N = k.m; q3.K = k.n; q3.tiles_n = k.m / PG_TILE;
            q3.A = k.QR; q3.lda = k.ldqr; q3.B = Np; q3.ldb = ldw; q3.C32 = Tt; q3.ldc32 = ldt;
            f3.push_back(q3);
            q.K = k.m; q.A = k.QL; q.lda = k.ldql; q.B = Tt; q.ldb = ldt; q.C32 = k.N; q.ldc32 = k.ldn; q.flags = 0;
            f4.push_back(q);
            tilesf += (k.m / PG_TILE) * q.tiles_n;
        } else {
            // 2: G' = Q_L^T (G Q_R):   A' = Q_L^T (m x m), B' = (G Q_R)^T (n x m)
            p.K = k.m; p.A = QLt; p.lda = ldqlt; p.B = Tt; p.ldb = ldt; p.C = Gr; p.ldc = ldw; p.flags = 0;
            p.tile_start = tiles;
            g2.push_back(p);
            // 3: (N' Q_R^T)^T:   A' = N' (m x n), B' = Q_R (B'(j, k) = Q_R[j][k]); stored transposed
            p.K = k.n; p.A = Np; p.lda = ldw; p.B = k.QR; p.ldb = k.ldqr; p.C = Tt; p.ldc = ldt; p.flags = GEMM_STORE_T;
            g3.push_back(p);
            // 4: N = Q_L (N' Q_R^T):   A' = Q_L (m x m), B' = (N' Q_R^T)^T (n x m)
            p.K = k.m; p.A = k.QL; p.lda = k.ldql; p.B = Tt; p.ldb = ldt; p.C = k.N; p.ldc = k.ldn; p.flags = 0;
            g4.push_back(p);
            tiles += tm * tn;
        }
        AdamBlock a;
        a.Gr = Gr; a.M = k.M; a.V = k.V; a.Np = Np; a.m = k.m; a.n = k.n; a.ldw = ldw; a.ldm = k.ldm; a.ldv = k.ldv;
        a.row_start = rows; rows += k.m;
        ab.push_back(a);
    }
    (void)tilesT;
    GemmProblem *d_g1b = d_g[0] + g1[0].size();
    // a two-sided block has one entry for its first product, of either kind: the region of d_g[0] holds them all
    static_assert(sizeof(PlaneProblem) <= sizeof(GemmProblem) && alignof(PlaneProblem) <= alignof(GemmProblem), "shared table region");
    PlaneProblem *d_f1 = reinterpret_cast<PlaneProblem *>(d_g1b + g1[1].size());
    Uploads up(stream);
    ASTERIA_HIP_TRY(up.add(d_g[0], g1[0].data(), g1[0].size() * sizeof(GemmProblem)));
    ASTERIA_HIP_TRY(up.add(d_g1b, g1[1].data(), g1[1].size() * sizeof(GemmProblem)));
    ASTERIA_HIP_TRY(up.add(d_f1, f1.data(), f1.size() * sizeof(PlaneProblem)));
    ASTERIA_HIP_TRY(up.add(d_g[1], g2.data(), g2.size() * sizeof(GemmProblem)));
    ASTERIA_HIP_TRY(up.add(d_g[2], g3.data(), g3.size() * sizeof(GemmProblem)));
    ASTERIA_HIP_TRY(up.add(d_g[3], g4.data(), g4.size() * sizeof(GemmProblem)));
    ASTERIA_HIP_TRY(up.add(d_f[0], f2.data(), f2.size() * sizeof(PlaneProblem)));
    ASTERIA_HIP_TRY(up.add(d_f[1], f3.data(), f3.size() * sizeof(PlaneProblem)));
    ASTERIA_HIP_TRY(up.add(d_f[2], f4.data(), f4.size() * sizeof(PlaneProblem)));
    ASTERIA_HIP_TRY(up.add(d_ab, ab.data(), ab.size() * sizeof(AdamBlock)));
    // tables of the one-sided blocks, one after the other in a region of their own
    GemmProblem *d_o = cv.take<GemmProblem>(4 * (size_t)nblocks);
    GemmProblem *d_oL1[2], *d_oR1[2], *d_oL2, *d_oR2;
    {
        GemmProblem *q = d_o;
        auto put = [&](const std::vector<GemmProblem> &v, GemmProblem *&dst) -> hipError_t {
            dst = q;
            q += v.size();
            return up.add(dst, v.data(), v.size() * sizeof(GemmProblem));
        };
        ASTERIA_HIP_TRY(put(oL1[0], d_oL1[0])); ASTERIA_HIP_TRY(put(oL1[1], d_oL1[1])); ASTERIA_HIP_TRY(put(oL2, d_oL2));
        ASTERIA_HIP_TRY(put(oR1[0], d_oR1[0])); ASTERIA_HIP_TRY(put(oR1[1], d_oR1[1])); ASTERIA_HIP_TRY(put(oR2, d_oR2));
    }
    ASTERIA_HIP_TRY(up.add(d_tj, tj.data(), tj.size() * sizeof(TransposeF32Job)));
    ASTERIA_HIP_TRY(up.flush());
    if (!tj.empty()) {
        hipLaunchKernelGGL(transpose_f32_kernel, dim3(ttiles), dim3(256), 0, stream, d_tj, (int)tj.size());
        ASTERIA_HIP_TRY(hipGetLastError());
    }
    // one-sided rotations into the eigenbasis
    ASTERIA_HIP_TRY((launch_gemm_grouped<float, float, float, true, true, true>(d_oL1[0], (int)oL1[0].size(), tL1[0], nullptr, stream)));
    ASTERIA_HIP_TRY((launch_gemm_grouped<float, float, bf16_t, true, true, true>(d_oL1[1], (int)oL1[1].size(), tL1[1], nullptr, stream)));
    ASTERIA_HIP_TRY((launch_gemm_grouped<float, float, float, false, true, true>(d_oR1[0], (int)oR1[0].size(), tR1[0], nullptr, stream)));
    ASTERIA_HIP_TRY((launch_gemm_grouped<float, bf16_t, float, false, true, true>(d_oR1[1], (int)oR1[1].size(), tR1[1], nullptr, stream)));
    if (!g1[0].empty())
        ASTERIA_HIP_TRY((launch_gemm_bf16_grouped<float, float, 2, 2>(d_g[0], (int)g1[0].size(), tiles1[0], nullptr, stream)));
    if (!g1[1].empty())
        ASTERIA_HIP_TRY((launch_gemm_bf16_grouped<bf16_t, float, 1, 2>(d_g1b, (int)g1[1].size(), tiles1[1], nullptr, stream)));
    if (!f1.empty()) ASTERIA_HIP_TRY((launch_pgemm<1>(d_f1, (int)f1.size(), tiles1f, stream, 514)));
    if (!g2.empty()) ASTERIA_HIP_TRY((launch_gemm_bf16_grouped<float, float, 2, 2>(d_g[1], (int)g2.size(), tiles, nullptr, stream)));
    if (!f2.empty()) ASTERIA_HIP_TRY((launch_pgemm<2>(d_f[0], (int)f2.size(), tilesf, stream, 513)));
    const float c1 = 1.0f - powf(beta1, (float)step_t), c2 = 1.0f - powf(beta2, (float)step_t);
    hipLaunchKernelGGL(adam_rotated_kernel, dim3(rows), dim3(256), 0, stream, d_ab, nblocks, beta1, beta2,
                       adam_eps, 1.0f / c1, 1.0f / c2);
    ASTERIA_HIP_TRY(hipGetLastError());
    if (!g2.empty()) ASTERIA_HIP_TRY((launch_gemm_bf16_grouped<float, float, 2, 2>(d_g[2], (int)g3.size(), tiles, nullptr, stream)));
    if (!f2.empty()) ASTERIA_HIP_TRY((launch_pgemm<2>(d_f[1], (int)f3.size(), tilesf, stream, 513)));
    if (!g2.empty()) ASTERIA_HIP_TRY((launch_gemm_bf16_grouped<float, float, 2, 2>(d_g[3], (int)g4.size(), tiles, nullptr, stream)));
    if (!f2.empty()) ASTERIA_HIP_TRY((launch_pgemm<2>(d_f[2], (int)f4.size(), tilesf, stream, 513)));
    // one-sided rotations back
    ASTERIA_HIP_TRY((launch_gemm_grouped<float, float, float, false, true, true>(d_oL2, (int)oL2.size(), tL2, nullptr, stream)));
    ASTERIA_HIP_TRY((launch_gemm_grouped<float, float, float, false, false, true>(d_oR2, (int)oR2.size(), tR2, nullptr, stream)));
    return ASTERIA_OK;
}

namespace {

// One region of a factor holds its projection coefficients and, between two projections, the partial Gram matrices of a
// panel and the fp32 inverse factor.  Several panels have coefficients at a time where a pass over the finished rows
// is shared: whole-panel factors with two panels beyond the first QR_AHEAD.
size_t refresh_scratch_bytes(int n, bool share)
{
    const size_t panels = share && n % QR_PANEL == 0 && n >= 2 * QR_AHEAD * QR_PANEL ? QR_AHEAD : 1;
    return std::max(Carver::need(panels * QR_PANEL * ld4(n), sizeof(float)),
                    Carver::need(gram_doubles(n), sizeof(double)) + Carver::need((size_t)QR_PANEL * QR_PANEL, sizeof(float)));
}

size_t refresh_factor_bytes(int n, bool share)
{
    const int np = (n + QR_PANEL - 1) / QR_PANEL;
    return Carver::need((size_t)n * ld4(n), sizeof(float)) +            // Z^T, becomes Q^T
           refresh_scratch_bytes(n, share) +
           Carver::need((size_t)n, sizeof(double)) + Carver::need((size_t)n, sizeof(int)) +   // column estimates and order
           (size_t)(1 + 2 * np) * sizeof(GemmProblem) + (size_t)(4 * np) * sizeof(PanelProblem) + (size_t)(np + 6) * sizeof(int) + sizeof(QrFactor);
}

// The factors of a call can be dealt to up to this many groups, each enqueued as a whole on an
// auxiliary stream the caller supplies (asteria_soap_refresh_overlapped); 4 groups: 328 ms against 318
// for 2 on the 1B-model workload (every group brings its own chain of launches).
constexpr int REFRESH_MAX_GROUPS = 4;

size_t refresh_fixed_bytes(int n_max)
{
    const int np = (n_max + QR_PANEL - 1) / QR_PANEL;
    return REFRESH_MAX_GROUPS * ((size_t)(5 * np + 4) * 256 + 4096);   // alignment slack of the per-panel tables, per group
}

// factors of a call from `first` on that one pass over it takes
int refresh_pass_count(const asteria_factor *f, int first, int nfactors, size_t fixed, size_t ws_bytes, bool share)
{
    size_t used = fixed;
    int cnt = 0;
    while (first + cnt < nfactors) {
        const size_t b = refresh_factor_bytes(f[first + cnt].n, share);
        if (used + b > ws_bytes) break;
        used += b;
        ++cnt;
    }
    return cnt;
}

// Whether panels share passes over the finished rows.  Their coefficients take 2 - 4 % of the workspace: they do unless the call
// would take more passes over its factors than without them, each a whole chain of panel steps; the sums of a factor and their
// order are the same either way.  Half of the factors' workspace without sharing, two passes without and three with it: 40
// factors of n = 1024 5.05 ms, 6.87; 12 of n = 2048 13.25, 17.6.
bool refresh_shares(const asteria_factor *f, int nfactors, size_t fixed, size_t ws_bytes)
{
    int passes[2] = {0, 0};
    for (int share = 0; share < 2; ++share)
        for (int first = 0; first < nfactors; ++passes[share]) {
            const int cnt = refresh_pass_count(f, first, nfactors, fixed, ws_bytes, share != 0);
            if (cnt == 0) return false;             // a factor that does not fit, or only without
            first += cnt;
        }
    return passes[1] <= passes[0];
}

}  // namespace

extern "C" size_t asteria_soap_refresh_workspace_bytes(const asteria_factor *f, int nfactors, size_t *min_bytes)
{
    if (min_bytes) *min_bytes = 0;
    if (!f || nfactors <= 0) return 0;
    size_t total = 0, biggest = 0;
    int n_max = 0;
    for (int i = 0; i < nfactors; ++i) {
        const int n = f[i].n;
        if (n <= 0) return 0;
        const size_t b = refresh_factor_bytes(n, false);
        total += refresh_factor_bytes(n, true);
        biggest = b > biggest ? b : biggest;
        n_max = n > n_max ? n : n_max;
    }
    if (min_bytes) *min_bytes = biggest + refresh_fixed_bytes(n_max);
    return total + refresh_fixed_bytes(n_max);
}

extern "C" asteria_status asteria_soap_refresh(const asteria_factor *f, int nfactors, int32_t *info,
                                               void *ws, size_t ws_bytes, void *stream_)
{
    return asteria_soap_refresh_ex(f, nfactors, nullptr, info, nullptr, ws, ws_bytes, stream_);
}

extern "C" void asteria_soap_refresh_opts_default(asteria_soap_refresh_opts *o)
{
    if (!o) return;
    o->sort = 0; o->from_identity = 0; o->rounds = 1; o->n_aux = 0; o->aux_streams = nullptr;
    o->Xt = nullptr; o->ldxt = nullptr; o->xt_in = 0;
}

extern "C" asteria_status asteria_soap_refresh_ex(const asteria_factor *f, int nfactors,
                                                  const asteria_soap_refresh_opts *opts_in, int32_t *info, int32_t *perm,
                                                  void *ws, size_t ws_bytes, void *stream_)
{
    if (!f || nfactors <= 0) return ASTERIA_INVALID_ARG;
    asteria_soap_refresh_opts o;
    asteria_soap_refresh_opts_default(&o);
    if (opts_in) o = *opts_in;
    if ((o.sort != 0 && o.sort != 1) || (o.from_identity != 0 && o.from_identity != 1) || o.rounds < 1 || o.rounds > 1000)
        return ASTERIA_INVALID_ARG;
    if (perm && (!o.sort || o.rounds != 1)) return ASTERIA_INVALID_ARG;   // the order of ONE sorted round can be reported
    if (o.xt_in != 0 && o.xt_in != 1) return ASTERIA_INVALID_ARG;
    if ((o.Xt != nullptr) != (o.ldxt != nullptr)) return ASTERIA_INVALID_ARG;
    void *const *aux_streams = o.aux_streams;
    const int n_aux = o.n_aux;
    if (n_aux < 0 || n_aux > REFRESH_MAX_GROUPS || (n_aux > 0 && !aux_streams)) return ASTERIA_INVALID_ARG;
    for (int g = 0; g < n_aux; ++g)
        if (!aux_streams[g] || aux_streams[g] == stream_) return ASTERIA_INVALID_ARG;
    int n_all = 0;
    for (int i = 0; i < nfactors; ++i) {
        if (!f[i].A || !f[i].X || f[i].n <= 0 || f[i].lda < f[i].n || f[i].ldx < f[i].n) return ASTERIA_INVALID_ARG;
        if (f[i].a_layout != ASTERIA_LAYOUT_FULL) return ASTERIA_UNSUPPORTED;   // A is an operand of the product A Q: full storage
        if (f[i].n > QR_MAXN) return ASTERIA_UNSUPPORTED;
        if (o.Xt && o.Xt[i] && (o.ldxt[i] < f[i].n || o.Xt[i] == f[i].X)) return ASTERIA_INVALID_ARG;
        n_all = f[i].n > n_all ? f[i].n : n_all;
    }
    if (!ws) return ASTERIA_WORKSPACE_TOO_SMALL;
    if (reinterpret_cast<uintptr_t>(ws) & 255u) return ASTERIA_INVALID_ARG;   // workspace must be 256-byte aligned
    // the first factor must fit: checked before anything touches the device
    if (refresh_fixed_bytes(n_all) + refresh_factor_bytes(f[0].n, false) > ws_bytes) return ASTERIA_WORKSPACE_TOO_SMALL;
    const bool share = refresh_shares(f, nfactors, refresh_fixed_bytes(n_all), ws_bytes);
    hipStream_t stream = reinterpret_cast<hipStream_t>(stream_);

    // the caller's permutation array holds the factors' orders one after the other
    std::vector<size_t> perm_offset(nfactors, 0);
    for (int i = 1; i < nfactors; ++i) perm_offset[i] = perm_offset[i - 1] + (size_t)f[i - 1].n;

    int first = 0;
    while (first < nfactors) {
        // largest pass that fits the workspace
        const int cnt = refresh_pass_count(f, first, nfactors, refresh_fixed_bytes(n_all), ws_bytes, share);
        if (cnt == 0) return ASTERIA_WORKSPACE_TOO_SMALL;
        // The factors of a pass are dealt to two groups, each enqueued as a whole on a stream of its
        // own: the panel steps of a group are a chain of small launches (projection, Gram matrix,
        // a latency-bound Cholesky kernel on one workgroup per factor, application), and two chains
        // running side by side fill the gaps each leaves on the device.
        Carver cv(ws);
        auto enqueue_group = [&](std::vector<int> idx, hipStream_t stream) -> asteria_status {
        const int cnt = (int)idx.size();
        if (cnt == 0) return ASTERIA_OK;
        // largest first: the factors that have panel j are then the first count[j] of the group
        std::stable_sort(idx.begin(), idx.end(), [&](int a, int b) { return f[a].n > f[b].n; });
        const int n_max = f[idx[0]].n;
        const int np_max = (n_max + QR_PANEL - 1) / QR_PANEL;

        QrFactor *d_q = cv.take<QrFactor>(cnt);
        std::vector<QrFactor> q;
        bool any_qt = false;                       // some factor's Q^T is kept by the caller
        // off | whole | pt | pp[0] | pp[1] | pz | slot: see RefreshTables
        std::vector<int> ints((size_t)(np_max + 1) + 4 * (size_t)(cnt + 1) + 2 * (size_t)cnt, 0);
        int *off = ints.data(), *nwhole = off + np_max + 1, *pt = nwhole + cnt + 1, *pp0 = pt + cnt + 1, *pp1 = pp0 + cnt + 1;
        int *pz = pp1 + cnt + 1, *slot = pz + cnt;
        std::vector<int> count(np_max, 0);
        for (int i = 0; i < cnt; ++i) {
            const asteria_factor &a = f[idx[i]];
            const int n = a.n, ldz = ld4(n);
            QrFactor F;
            memset(&F, 0, sizeof(F));
            F.Zt = cv.take<float>((size_t)n * ldz);
            unsigned char *scratch = cv.take<unsigned char>(refresh_scratch_bytes(n, share));
            F.cbuf = reinterpret_cast<float *>(scratch);
            F.gram = reinterpret_cast<double *>(scratch);
            F.winv = reinterpret_cast<float *>(scratch + Carver::need(gram_doubles(n), sizeof(double)));
            F.Qout = a.X; F.n = n; F.ldz = ldz; F.ldq = a.ldx; F.bad = 0; F.run = 0; F.skip3 = 1;
            F.out_index = idx[i];
            F.Qt = a.X; F.ldqt = a.ldx;
            if (o.Xt && o.Xt[idx[i]]) { F.Qt = o.Xt[idx[i]]; F.ldqt = o.ldxt[idx[i]]; any_qt = true; }
            F.a_scale = 1.0f; F.p_scale = 1.0f; F.A = a.A; F.lda = a.lda;
            F.est = cv.take<double>((size_t)n);
            F.perm = cv.take<int>((size_t)n);
            F.perm_out = perm ? perm + perm_offset[idx[i]] : nullptr;
            q.push_back(F);
            const int tn = (n + BN - 1) / BN;
            const bool panels = n % QR_PANEL == 0 && (a.ldx & 3) == 0 && (reinterpret_cast<uintptr_t>(a.X) & 15u) == 0;
            nwhole[i + 1] = nwhole[i] + (panels ? 1 : 0);
            pt[i + 1] = pt[i] + (panels ? 0 : tn);
            pp0[i + 1] = pp0[i] + (panels ? tn : 0);
            pp1[i + 1] = pp1[i] + (panels ? (tn + 1) / 2 : 0);
            for (int j = 0; j < (n + QR_PANEL - 1) / QR_PANEL; ++j) ++count[j];
        }
        for (int j = 0; j < np_max; ++j) off[j + 1] = off[j] + count[j];
        // The Z products of whole-tile factors run on the kernel of pgemm.h and the others on that of gemm_bf16.h, whose sums have
        // another order: by the factor alone, so that its result does not depend on what it is batched with.  Only the
        // width of the tiles goes by the group: large ones beyond 128, where small ones need a second round of the chip (two
        // workgroups a CU), but not where a few of them would need a second round of their own (one a CU).  Product in us, small /
        // large tiles, by large ones: n = 256 64 19 / 28, 128: 26 / 31, 192: 36 / 35, 256: 48 / 40, 264: 50 / 58, 320: 60 / 63, 340: 66 / 65, 512:
        // 98 / 85; n = 512 128 37 / 44, 160: 48 / 46, 256: 64 / 55, 280: 78 / 86, 320: 87 / 91, 340: 97 / 92; n = 1024 64 40 / 70, 128: 60 / 75,
        // 160: 83 / 77, 256: 111 / 91, 272: 130 / 146, 320: 138 / 151, 336: 155 / 153, 384: 170 / 159, 512: 220 / 180; n = 2048 128 109 / 136, 192:
        // 162 / 148, 320: 259 / 278, 512: 413 / 332.  (Small tiles of gemm_bf16.h: n = 1024 64 47, 128: 65.)
        auto whole = [](const QrFactor &F, int edge) {
            return pg_f32_operand_ok(F.Qt, F.n, F.n, F.ldqt, edge) && pg_f32_operand_ok(F.A, F.n, F.n, F.lda, edge);
        };
        long long large_tiles = 0;
        int large = 0;
        for (const QrFactor &F : q)
            if (whole(F, PG_TILE)) {
                large_tiles += (long long)(F.n / PG_TILE) * (F.n / PG_TILE);
                ++large;
            }
        if (large_tiles <= 128 || (large_tiles > 256 && large_tiles <= 320)) large = 0;
        int nz = 0, nl = 0, ns = large, tiles = 0, tiles_l = 0, tiles_s = 0;
        for (int i = 0; i < cnt; ++i) {
            const int n = q[i].n, tn = (n + BN - 1) / BN;
            if (large && whole(q[i], PG_TILE)) {
                slot[i] = -1 - nl++;
                pz[i] = tiles_l;
                tiles_l += (n / PG_TILE) * (n / PG_TILE);
            } else if (whole(q[i], PG_SMALL_TILE)) {
                slot[i] = -1 - ns++;
                pz[i] = tiles_s;
                tiles_s += (n / PG_SMALL_TILE) * (n / PG_SMALL_TILE);
            } else {
                slot[i] = nz++;
                pz[i] = tiles;
                tiles += tn * tn;
            }
        }
        const int entries = off[np_max];
        RefreshTables rt;
        rt.z = cv.take<GemmProblem>(nz);
        rt.zp = cv.take<PlaneProblem>(ns);
        rt.zp_large = large;
        rt.t1 = cv.take<GemmProblem>(entries); rt.t2 = cv.take<GemmProblem>(entries);
        rt.f1 = cv.take<PanelProblem>(entries); rt.f2 = cv.take<PanelProblem>(entries);
        rt.p1 = cv.take<PanelProblem>(entries); rt.p2 = cv.take<PanelProblem>(entries);
        int *d_ints = cv.take<int>(ints.size());
        rt.off = d_ints; rt.whole = d_ints + (nwhole - off); rt.pt = d_ints + (pt - off);
        rt.pp[0] = d_ints + (pp0 - off); rt.pp[1] = d_ints + (pp1 - off);
        rt.pz = d_ints + (pz - off); rt.slot = d_ints + (slot - off);
        rt.share = share ? 1 : 0;
        Uploads up(stream);
        ASTERIA_HIP_TRY(up.add(d_q, q.data(), q.size() * sizeof(QrFactor)));
        ASTERIA_HIP_TRY(up.add(d_ints, ints.data(), ints.size() * sizeof(int)));
        ASTERIA_HIP_TRY(up.flush());
        hipLaunchKernelGGL(refresh_tables_kernel, dim3((cnt + 127) / 128, np_max), dim3(128), 0, stream, d_q, cnt, rt);
        ASTERIA_HIP_TRY(hipGetLastError());
        // the two products of a projection of panel j, with `ny` fp16 terms of the panel's rows (and as many of the
        // finished rows in the first) and `nx` of the finished rows in the second
        auto project = [&](int j, auto ny_, auto nx_, const int *st) -> asteria_status {
            constexpr int NY = decltype(ny_)::value, NX = decltype(nx_)::value;
            const int c = count[j], w = nwhole[c];
            // the factors with a remainder have all of theirs in the last call for the whole panels
            GemmProblem *t1 = rt.t1 + off[j], *t2 = rt.t2 + off[j];
            const int ragged1 = (c - w) * j, ragged2 = pt[c];
            // whole panels: `slots` of them against `rows` panels of finished rows
            auto panels = [&](const PanelProblem *p1, const PanelProblem *p2, int rows, int slots, bool with_ragged) -> asteria_status {
                const int narrow1 = w * rows * slots, wide1 = w * ((rows + 1) / 2) * slots, narrow2 = pp0[c] * slots, wide2 = pp1[c] * slots;
                if (with_ragged && w > 0 && w < c) {
                    if (pp_take_wide_tiles(wide1)) ASTERIA_HIP_TRY((launch_joint_product<NY, NY, 4>(p1, c, wide1, t1, c, ragged1, st, stream)));
                    else ASTERIA_HIP_TRY((launch_joint_product<NY, NY, 2>(p1, c, narrow1, t1, c, ragged1, st, stream)));
                    if (pp_take_wide_tiles(wide2)) ASTERIA_HIP_TRY((launch_joint_product<NY, NX, 4>(p2, c, wide2, t2, c, ragged2, st, stream)));
                    else ASTERIA_HIP_TRY((launch_joint_product<NY, NX, 2>(p2, c, narrow2, t2, c, ragged2, st, stream)));
                    return ASTERIA_OK;
                }
                if (with_ragged) {
                    ASTERIA_HIP_TRY((launch_gemm_bf16_grouped<float, float, NY, NY, true>(t1, c, ragged1, st, stream)));
                    ASTERIA_HIP_TRY((launch_gemm_bf16_grouped<float, float, NY, NX, true>(t2, c, ragged2, st, stream)));
                }
                if (pp_take_wide_tiles(wide1)) ASTERIA_HIP_TRY((launch_panel_product<NY, NY, 4>(p1, c, wide1, st, stream)));
                else ASTERIA_HIP_TRY((launch_panel_product<NY, NY, 2>(p1, c, narrow1, st, stream)));
                if (pp_take_wide_tiles(wide2)) ASTERIA_HIP_TRY((launch_panel_product<NY, NX, 4>(p2, c, wide2, st, stream)));
                else ASTERIA_HIP_TRY((launch_panel_product<NY, NX, 2>(p2, c, narrow2, st, stream)));
                return ASTERIA_OK;
            };
            const int near = NY == 1 ? j % QR_AHEAD : 0, far = j - near;
            if (near == 0) {
                if (NY == 1 && share) return panels(rt.f1 + off[j], rt.f2 + off[j], j, std::min(QR_AHEAD, np_max - j), true);
                return panels(rt.p1 + off[j], rt.p2 + off[j], j, 1, true);
            }
            if (!share && far > 0)
                if (const asteria_status ps = panels(rt.f1 + off[far], rt.f2 + off[far], far, 1, false); ps != ASTERIA_OK) return ps;
            return panels(rt.f1 + off[j], rt.f2 + off[j], near, 1, true);
        };
        hipLaunchKernelGGL(qr_scale_kernel, dim3(cnt), dim3(64), 0, stream, d_q, cnt);
        if (o.from_identity)
            hipLaunchKernelGGL(set_identity_kernel, dim3((unsigned)std::min<size_t>(((size_t)n_max * n_max + 255) / 256, 4096), (unsigned)cnt),
                               dim3(256), 0, stream, d_q);
        const unsigned tpr32 = (unsigned)((n_max + 31) / 32);
        // a kept Q^T that the caller has not filled (or a start from the identity, which the kernel above
        // wrote to both buffers) is made from Q once; every round then leaves the new one there
        if (any_qt && !o.xt_in && !o.from_identity)
            hipLaunchKernelGGL(keep_qt_kernel, dim3(tpr32 * tpr32, (unsigned)cnt), dim3(256), 0, stream, d_q);
        for (int round = 0; round < o.rounds; ++round) {
        hipLaunchKernelGGL(transpose_inplace_kernel, dim3(tpr32 * tpr32, (unsigned)cnt), dim3(256), 0, stream, d_q);
        ASTERIA_HIP_TRY((launch_pgemm<2, true>(rt.zp, large, tiles_l, stream, 513)));
        ASTERIA_HIP_TRY(launch_product_f16(rt.zp + large, ns - large, tiles_s, rt.z, nz, tiles, stream));
        if (o.sort) {
            // order the columns by q_i^T A q_i = (row i of Q^T) . (row i of Z^T), largest first: the rows of
            // Z^T are gathered in that order (A (Q P) = (A Q) P: sorting the basis first, as SOAP does, and
            // then multiplying gives the same Z)
            hipLaunchKernelGGL(sort_estimate_kernel, dim3((unsigned)((n_max + 3) / 4), (unsigned)cnt), dim3(256), 0, stream, d_q);
            hipLaunchKernelGGL(sort_rank_kernel, dim3((unsigned)((n_max + RANK_COLS - 1) / RANK_COLS), (unsigned)cnt), dim3(256), 0, stream, d_q);
            hipLaunchKernelGGL(sort_gather_kernel, dim3((unsigned)n_max, (unsigned)cnt), dim3(256), 0, stream, d_q, 0);
            hipLaunchKernelGGL(sort_gather_kernel, dim3((unsigned)n_max, (unsigned)cnt), dim3(256), 0, stream, d_q, 1);
            ASTERIA_HIP_TRY(hipGetLastError());
        }
        for (int j = 0; j < np_max; ++j) {
            // sweeps of (project against the finished rows, orthonormalise the panel): the second
            // projection acts on normalised rows, so what the first normalisation amplified - the
            // residue of the first projection, O(1) for a row that was numerically dependent - is
            // removed again and a rank-deficient A Q still yields an orthogonal Q; factors in which
            // the second sweep met such a row run a third one
            const int *st_run = reinterpret_cast<const int *>(d_q) + offsetof(QrFactor, run) / sizeof(int);
            const int *st_third = reinterpret_cast<const int *>(d_q) + offsetof(QrFactor, skip3) / sizeof(int);
            for (int sweep = 0; sweep < 3; ++sweep) {
                const int *st = sweep < 2 ? st_run : st_third;
                if (j > 0) {
                    // projection coefficients: fp32 operands as two fp16 terms each (2^-22) in the second
                    // sweep and in the third, which only the factors that need it run (their rows are still
                    // normalised there: the Cholesky kernel keeps the unit scale until a panel's last sweep)
                    // first sweep: the coefficients as one fp16 term per operand, and one term of them in
                    // the update (the finished rows keep both terms, so the panel stays in the span of
                    // its own rows and the finished ones to 2^-22): what this leaves along the finished
                    // rows, 2^-11 of the coefficients, is what the second sweep removes at full accuracy
                    using One = std::integral_constant<int, 1>;
                    using Two = std::integral_constant<int, 2>;
                    const asteria_status ps = sweep == 0 ? project(j, One{}, Two{}, st) : project(j, Two{}, Two{}, st);
                    if (ps != ASTERIA_OK) return ps;
                }
                const unsigned nfac = (unsigned)count[j];
                hipLaunchKernelGGL(panel_gram_kernel, dim3((unsigned)gram_splits(n_max), nfac), dim3(256), 0, stream, d_q, j, sweep);
                hipLaunchKernelGGL(panel_chol_kernel, dim3(nfac), dim3(256), 0, stream, d_q, j, sweep);
                hipLaunchKernelGGL(panel_apply_kernel, dim3((unsigned)((n_max + 127) / 128), nfac), dim3(256), 0, stream, d_q, j, sweep);
                ASTERIA_HIP_TRY(hipGetLastError());
            }
        }
        }   // rounds
        hipLaunchKernelGGL(qr_info_kernel, dim3((cnt + 127) / 128), dim3(128), 0, stream, d_q, cnt, info);
        ASTERIA_HIP_TRY(hipGetLastError());
        return ASTERIA_OK;
        };
        if (n_aux < 2 || cnt < n_aux) {
            std::vector<int> all(cnt);
            for (int i = 0; i < cnt; ++i) all[i] = first + i;
            hipStream_t s0 = (n_aux == 1) ? reinterpret_cast<hipStream_t>(aux_streams[0]) : stream;
            hipEvent_t fork = nullptr, join = nullptr;
            if (n_aux == 1) {
                ASTERIA_HIP_TRY(hipEventCreateWithFlags(&fork, hipEventDisableTiming));
                ASTERIA_HIP_TRY(hipEventCreateWithFlags(&join, hipEventDisableTiming));
                ASTERIA_HIP_TRY(hipEventRecord(fork, stream));
                ASTERIA_HIP_TRY(hipStreamWaitEvent(s0, fork, 0));
            }
            const asteria_status st = enqueue_group(all, s0);
            if (n_aux == 1) {
                if (st == ASTERIA_OK) {
                    ASTERIA_HIP_TRY(hipEventRecord(join, s0));
                    ASTERIA_HIP_TRY(hipStreamWaitEvent(stream, join, 0));
                }
                (void)hipEventDestroy(fork);        // released once the recorded work has passed them
                (void)hipEventDestroy(join);
            }
            if (st != ASTERIA_OK) return st;
        } else {
            // fork: every auxiliary stream starts after everything already enqueued on the caller's
            // stream (the previous pass included); join: the caller's stream continues after all of
            // them.  The events live for this call only (destroying a recorded event releases it once
            // the work it marks has completed).
            std::vector<std::vector<int>> grp(n_aux);
            for (int i = 0; i < cnt; ++i) grp[i % n_aux].push_back(first + i);
            hipEvent_t fork = nullptr;
            ASTERIA_HIP_TRY(hipEventCreateWithFlags(&fork, hipEventDisableTiming));
            ASTERIA_HIP_TRY(hipEventRecord(fork, stream));
            asteria_status st = ASTERIA_OK;
            for (int g2 = 0; g2 < n_aux && st == ASTERIA_OK; ++g2) {
                hipStream_t sg = reinterpret_cast<hipStream_t>(aux_streams[g2]);
                hipEvent_t join = nullptr;
                if (hipEventCreateWithFlags(&join, hipEventDisableTiming) != hipSuccess ||
                    hipStreamWaitEvent(sg, fork, 0) != hipSuccess) {
                    if (join) (void)hipEventDestroy(join);
                    st = ASTERIA_HIP_ERROR;
                    break;
                }
                st = enqueue_group(grp[g2], sg);
                if (st == ASTERIA_OK && (hipEventRecord(join, sg) != hipSuccess ||
                                         hipStreamWaitEvent(stream, join, 0) != hipSuccess)) st = ASTERIA_HIP_ERROR;
                (void)hipEventDestroy(join);
            }
            (void)hipEventDestroy(fork);
            if (st != ASTERIA_OK) return st;
        }

        first += cnt;
    }
    return ASTERIA_OK;
}

// ---------------------------------------------------------------------------------------------
// asteria_soap_reproject: the first moment M of asteria_soap_step lives in the rotated space of the
// bases it was accumulated in.  When a refresh replaces (Q_L, Q_R), the matrix M stands for in the
// original space, W = Q_L,old M Q_R,old^T, is re-expressed in the new bases: M <- Q_L,new^T W Q_R,new.
// Four grouped products on the bf16 matrix cores with two-term split operands, as in
// asteria_soap_step.  The second moment V is not a linear quantity; it follows the column order only
// (V[i][j] <- V[permL[i]][permR[j]], the orders a sorted refresh reports).
namespace {

struct PermuteJob {
    float *V;          // m x n, ldv
    float *tmp;        // m x n, ldw
    const int *pl, *pr;   // row / column order, or null for the identity
    int m, n, ldv, ldw;
    int row_start;
    int pad_;
};

__global__ __launch_bounds__(256) void permute_moment_kernel(const PermuteJob *jobs, int njobs, int phase)
{
    int lo = 0, hi = njobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (jobs[mid].row_start <= (int)blockIdx.x) lo = mid; else hi = mid - 1;
    }
    const PermuteJob &J = jobs[lo];
    const int i = (int)blockIdx.x - J.row_start;
    if (phase == 0) {
        const float *src = J.V + (size_t)(J.pl ? J.pl[i] : i) * J.ldv;
        float *dst = J.tmp + (size_t)i * J.ldw;
        for (int j = threadIdx.x; j < J.n; j += 256) dst[j] = src[J.pr ? J.pr[j] : j];
    } else {
        const float *src = J.tmp + (size_t)i * J.ldw;
        float *dst = J.V + (size_t)i * J.ldv;
        for (int j = threadIdx.x; j < J.n; j += 256) dst[j] = src[j];
    }
}

asteria_status validate_reproject(const asteria_rblock *b, int nblocks)
{
    if (!b || nblocks <= 0) return ASTERIA_INVALID_ARG;
    for (int i = 0; i < nblocks; ++i) {
        const asteria_rblock &k = b[i];
        if (k.m <= 0 || k.n <= 0) return ASTERIA_INVALID_ARG;
        if (!k.M && !k.V) return ASTERIA_INVALID_ARG;
        if (k.M && (!k.QL_old || !k.QL_new || !k.QR_old || !k.QR_new)) return ASTERIA_INVALID_ARG;
        if (k.M && (k.ldql_old < k.m || k.ldql_new < k.m || k.ldqr_old < k.n || k.ldqr_new < k.n || k.ldm < k.n))
            return ASTERIA_INVALID_ARG;
        if (k.V && k.ldv < k.n) return ASTERIA_INVALID_ARG;
    }
    return ASTERIA_OK;
}

}  // namespace

extern "C" size_t asteria_soap_reproject_workspace_bytes(const asteria_rblock *blocks, int nblocks)
{
    if (!blocks || nblocks <= 0) return 0;
    size_t bytes = 4 * Carver::need((size_t)nblocks, sizeof(GemmProblem)) + Carver::need((size_t)nblocks, sizeof(PermuteJob)) +
                   Carver::need(2 * (size_t)nblocks, sizeof(TransposeF32Job)) + 2048;
    for (int i = 0; i < nblocks; ++i) {
        const int m = blocks[i].m, n = blocks[i].n;
        bytes += Carver::need((size_t)m * ld4(n), sizeof(float));          // W, also the copy of V while it is permuted
        bytes += Carver::need((size_t)n * ld4(m), sizeof(float));          // transposed intermediate (n x m)
        bytes += Carver::need((size_t)m * ld4(m), sizeof(float));          // Q_L,new^T
        bytes += Carver::need((size_t)n * ld4(n), sizeof(float));          // Q_R,new^T
    }
    return bytes;
}

extern "C" asteria_status asteria_soap_reproject(const asteria_rblock *blocks, int nblocks,
                                                 void *ws, size_t ws_bytes, void *stream_)
{
    asteria_status st = validate_reproject(blocks, nblocks);
    if (st != ASTERIA_OK) return st;
    if (!ws || ws_bytes < asteria_soap_reproject_workspace_bytes(blocks, nblocks)) return ASTERIA_WORKSPACE_TOO_SMALL;
    if (reinterpret_cast<uintptr_t>(ws) & 255u) return ASTERIA_INVALID_ARG;
    hipStream_t stream = reinterpret_cast<hipStream_t>(stream_);

    Carver cv(ws);
    GemmProblem *d_g[4];
    for (int i = 0; i < 4; ++i) d_g[i] = cv.take<GemmProblem>(nblocks);
    PermuteJob *d_pj = cv.take<PermuteJob>(nblocks);
    TransposeF32Job *d_tj = cv.take<TransposeF32Job>(2 * (size_t)nblocks);
    std::vector<GemmProblem> g[4];
    std::vector<PermuteJob> pj;
    std::vector<TransposeF32Job> tj;
    int tiles = 0, ttiles = 0, prow = 0;
    for (int i = 0; i < nblocks; ++i) {
        const asteria_rblock &k = blocks[i];
        const int ldw = ld4(k.n), ldt = ld4(k.m), ldqlt = ld4(k.m), ldqrt = ld4(k.n);
        float *Wb = cv.take<float>((size_t)k.m * ldw);
        float *Tt = cv.take<float>((size_t)k.n * ldt);
        float *QLt = cv.take<float>((size_t)k.m * ldqlt);
        float *QRt = cv.take<float>((size_t)k.n * ldqrt);
        if (k.V && (k.permL || k.permR)) {
            PermuteJob j;
            memset(&j, 0, sizeof(j));
            j.V = k.V; j.tmp = Wb; j.pl = k.permL; j.pr = k.permR; j.m = k.m; j.n = k.n; j.ldv = k.ldv; j.ldw = ldw;
            j.row_start = prow; prow += k.m;
            pj.push_back(j);
        }
        if (!k.M) continue;
        TransposeF32Job t;
        memset(&t, 0, sizeof(t));
        t.src = k.QL_new; t.dst = QLt; t.rows = k.m; t.cols = k.m; t.lds_ = k.ldql_new; t.ldd = ldqlt;
        t.tile_start = ttiles; ttiles += ((k.m + 31) / 32) * ((k.m + 31) / 32);
        tj.push_back(t);
        t.src = k.QR_new; t.dst = QRt; t.rows = k.n; t.cols = k.n; t.lds_ = k.ldqr_new; t.ldd = ldqrt;
        t.tile_start = ttiles; ttiles += ((k.n + 31) / 32) * ((k.n + 31) / 32);
        tj.push_back(t);
        const int tm = (k.m + BM - 1) / BM, tn = (k.n + BN - 1) / BN;
        GemmProblem p;
        memset(&p, 0, sizeof(p));
        p.state_idx = -1; p.state_mask = ~0; p.alpha = 1.0f; p.beta = 0.0f;
        p.M = k.m; p.N = k.n; p.tiles_n = tn; p.tile_start = tiles;
        // a: (M Q_R,old^T)^T:  A' = M, B'(j, k) = Q_R,old[j][k]; stored transposed
        p.K = k.n; p.A = k.M; p.lda = k.ldm; p.B = k.QR_old; p.ldb = k.ldqr_old; p.C = Tt; p.ldc = ldt; p.flags = GEMM_STORE_T;
        g[0].push_back(p);
        // b: W = Q_L,old (M Q_R,old^T):  A' = Q_L,old, B' = the transposed intermediate
        p.K = k.m; p.A = k.QL_old; p.lda = k.ldql_old; p.B = Tt; p.ldb = ldt; p.C = Wb; p.ldc = ldw; p.flags = 0;
        g[1].push_back(p);
        // c: (W Q_R,new)^T:  A' = W, B'(j, k) = Q_R,new[k][j] = its transposed copy; stored transposed
        p.K = k.n; p.A = Wb; p.lda = ldw; p.B = QRt; p.ldb = ldqrt; p.C = Tt; p.ldc = ldt; p.flags = GEMM_STORE_T;
        g[2].push_back(p);
        // d: M = Q_L,new^T (W Q_R,new):  A' = Q_L,new^T, B' = the transposed intermediate
        p.K = k.m; p.A = QLt; p.lda = ldqlt; p.B = Tt; p.ldb = ldt; p.C = k.M; p.ldc = k.ldm; p.flags = 0;
        g[3].push_back(p);
        tiles += tm * tn;
    }
    Uploads up(stream);
    ASTERIA_HIP_TRY(up.add(d_pj, pj.data(), pj.size() * sizeof(PermuteJob)));
    ASTERIA_HIP_TRY(up.add(d_tj, tj.data(), tj.size() * sizeof(TransposeF32Job)));
    for (int i = 0; i < 4; ++i) ASTERIA_HIP_TRY(up.add(d_g[i], g[i].data(), g[i].size() * sizeof(GemmProblem)));
    ASTERIA_HIP_TRY(up.flush());
    // V first: its copy uses the W buffer of the block
    if (!pj.empty()) {
        for (int phase = 0; phase < 2; ++phase)
            hipLaunchKernelGGL(permute_moment_kernel, dim3(prow), dim3(256), 0, stream, d_pj, (int)pj.size(), phase);
        ASTERIA_HIP_TRY(hipGetLastError());
    }
    if (g[0].empty()) return ASTERIA_OK;
    hipLaunchKernelGGL(transpose_f32_kernel, dim3(ttiles), dim3(256), 0, stream, d_tj, (int)tj.size());
    ASTERIA_HIP_TRY(hipGetLastError());
    for (int i = 0; i < 4; ++i)
        ASTERIA_HIP_TRY((launch_gemm_bf16_grouped<float, float, 2, 2>(d_g[i], (int)g[i].size(), tiles, nullptr, stream)));
    return ASTERIA_OK;
}
