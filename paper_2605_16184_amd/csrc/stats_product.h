// L <- beta L + (1 - beta) G G^T and R <- beta R + (1 - beta) G^T G of bf16 gradients on the bf16 matrix cores.
#pragma once
#include <type_traits>

#include "planes.h"

namespace asteria {

typedef __bf16 st_bf16x8 __attribute__((ext_vector_type(8)));

// One gradient block with the statistics this launch updates (null: not this one).
struct StatsEntry {
    const uint16_t *G;      // m x n, or n x m (transposed copy) when STATS_TRANSPOSED: then only R is updated
    float *L, *R;
    int m, n, ldg, ldl, ldr;
    int flags;
    int tile_start;         // first tile of the entry in the launch: those of L, then those of R
    int pad_;
};
enum : int { STATS_TRANSPOSED = 1, STATS_PACKED = 2 };

// Operands the kernel reads in place: 16-byte aligned rows of whole 16-byte pieces, offsets within 31 bits
inline bool stats_operand_ok(const void *p, int rows, int cols, int ld)
{
    return (reinterpret_cast<uintptr_t>(p) & 15u) == 0 && (ld % 8) == 0 && (cols % 8) == 0 && (size_t)rows * (size_t)ld * 2 < 0x70000000u;
}

// ST: slabs of LDS; with two the next slab is on its way while one is multiplied.
// The K loop: acc += A B^T over the rows row0 .. and col0 .. of an operand of n rows (columns when KM), K long.
template <bool KM, int ST>
__device__ __forceinline__ void stats_k_loop(floatx16 (&acc)[2][2], const uint16_t *G, int ldg, int n, int K, int row0, int col0,
                                             ASTERIA_LDS char *lds, int wave, int lane)
{
    constexpr int OP = 128 * 128;                             // bytes of an operand's slab
    const bool diag = row0 == col0;
    ASTERIA_LDS char *const first = lds;
    const int wm = wave >> 1, wn = wave & 1, r = lane & 31, h = lane >> 5;
    // wavefront w stages instructions 4 w .. 4 w + 3 of each operand's 16 (64 chunks of 16 bytes each)
    constexpr uint32_t OUTSIDE = 0x7ffffff0u;
    const uint32_t ldb = (uint32_t)ldg * 2u;
    const i32x4 rs = buffer_rsrc(G, (uint32_t)((KM ? K : n) - 1) * ldb + (uint32_t)(KM ? n : (K + 7) / 8 * 8) * 2u);   // whole pieces: a copy is padded
    uint32_t va[4], vb[4];
    int kof[4];                                               // k of the chunk within the slab
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int p = (wave * 4 + v) * 64 + lane;
        if constexpr (KM) {
            const int k = p >> 4, c16 = p & 15, c = ((((c16 >> 2) ^ (k & 3)) << 2) | (c16 & 3)) * 8;
            kof[v] = k;
            va[v] = (uint32_t)k * ldb + (uint32_t)min(row0 + c, n - 8) * 2u;
            vb[v] = (uint32_t)k * ldb + (uint32_t)min(col0 + c, n - 8) * 2u;
        } else {
            const int rr = p >> 3, c = ((p & 7) ^ plane_swz<8>(rr)) * 8;
            kof[v] = c;
            va[v] = (uint32_t)min(row0 + rr, n - 1) * ldb + (uint32_t)c * 2u;
            vb[v] = (uint32_t)min(col0 + rr, n - 1) * ldb + (uint32_t)c * 2u;
        }
    }
    const uint32_t slab_bytes = KM ? 64u * ldb : 128u;
    const uint32_t lds_first = (uint32_t)(uintptr_t)lds + (uint32_t)wave * 4096u;
    auto issue = [&](int slab) __attribute__((always_inline)) {
        const uint32_t off = (uint32_t)slab * slab_bytes, lds0 = lds_first + (uint32_t)(slab & (ST - 1)) * (2u * OP);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const bool in = slab * 64 + kof[v] < K;
            load_to_lds(rs, lds0 + (uint32_t)v * 1024u, in ? va[v] + off : OUTSIDE, 0u);
            if (!diag) load_to_lds(rs, lds0 + OP + (uint32_t)v * 1024u, in ? vb[v] + off : OUTSIDE, 0u);
        }
    };
    const int nk = (K + 63) / 64;
    const uint32_t bo = diag ? 0u : (uint32_t)OP;
    const int diag_d = diag ? wm - wn : 1;                    // < 0: above the diagonal, 0: on it
    auto multiply = [&](const u32x4 (&af)[2], const u32x4 (&bf)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                if (!(i == 0 && j == 1 && diag_d == 0))
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(st_bf16x8, af[i]), __builtin_bit_cast(st_bf16x8, bf[j]),
                                                                        acc[i][j], 0, 0, 0);
    };
    uint32_t fa[2], fb[2];
    const int sw = plane_swz<8>(r);
    {
        const int g = lane >> 4, e = (lane >> 2) & 3, q = lane & 3;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if constexpr (KM) {
                const uint32_t rc = (uint32_t)((8 * (g >> 1) + e) * 256 + (16 * (g & 1) + 4 * q) * 2);
                fa[i] = rc + ((uint32_t)((wm * 2 + i) ^ e) << 6);
                fb[i] = bo + rc + ((uint32_t)((wn * 2 + i) ^ e) << 6);
            } else {
                fa[i] = (uint32_t)((wm * 64 + i * 32 + r) * 128);
                fb[i] = bo + (uint32_t)((wn * 64 + i * 32 + r) * 128);
            }
        }
    }
    auto compute = [&]() __attribute__((always_inline)) {
        if constexpr (KM) {
            auto frag = [&](uint32_t off) __attribute__((always_inline)) {
                typedef short s16x4 __attribute__((ext_vector_type(4)));
                typedef uint32_t u2 __attribute__((ext_vector_type(2)));
                const u2 a = __builtin_bit_cast(u2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((ASTERIA_LDS s16x4 *)(lds + off)));
                const u2 b = __builtin_bit_cast(u2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((ASTERIA_LDS s16x4 *)(lds + off + 1024)));
                return (u32x4){a[0], a[1], b[0], b[1]};
            };
            u32x4 af[2][2], bf[2][2];
            auto read = [&](int s) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < 2; ++i) { af[s & 1][i] = frag(fa[i] + s * 4096); bf[s & 1][i] = frag(fb[i] + s * 4096); }
            };
            read(0);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                if (s < 3) read(s + 1);
                __builtin_amdgcn_sched_barrier(0);        // the fragments of one step ahead: four would spill
                multiply(af[s & 1], bf[s & 1]);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            u32x4 af[2][2], bf[2][2];
            auto read = [&](int s) __attribute__((always_inline)) {
                const uint32_t c = (uint32_t)(((s * 2 + h) ^ sw) * 16);
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    af[s & 1][i] = *(const ASTERIA_LDS u32x4 *)(lds + fa[i] + c);
                    bf[s & 1][i] = *(const ASTERIA_LDS u32x4 *)(lds + fb[i] + c);
                }
            };
            read(0);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                if (s < 3) read(s + 1);
                __builtin_amdgcn_sched_barrier(0);
                multiply(af[s & 1], bf[s & 1]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    if (ST == 2) issue(0);
    for (int kt = 0; kt < nk; ++kt) {
        if (ST == 1) issue(kt);
        if (ST == 2 && kt + 1 < nk) {
            issue(kt + 1);
            if (diag) wait_lds_loads<4>(); else wait_lds_loads<8>();
        } else wait_lds_loads<0>();
        lds = first + (kt & (ST - 1)) * (2 * OP);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");                        // the reads stay behind the barrier
        if (diag_d >= 0) compute();
        if (ST == 1) wait_lds_loads<0>();                     // this wavefront has read the slab
        else asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
    }
}

// A 128 x 128 tile of a symmetric product per workgroup, 2 x 2 wavefronts of 2 x 2 MFMA blocks, slabs of 64 k.
//   G G^T: both operands k-contiguous, LDS rows of 128 bytes.  G^T G: both k-major, LDS row = k, 256 bytes; the
//   MFMA operands (8 consecutive k of one column per lane) come out through ds_read_b64_tr_b16, which transposes
//   within 16 lanes: lane 4 e + q supplies the address of elements 4 q .. 4 q + 3 of row k0 + e, and lane j
//   receives element j of rows k0 .. k0 + 3.
// Operands go from memory to LDS without registers; rows and columns beyond the matrix repeat the last one (never
// stored), k beyond its end reads as zero through the bounds check of the buffer loads.
//
// At n = 1024 a tile moves 128 KiB of statistics (256 in full storage) for 34 MFLOP, so both pipes matter and the
// epilogue has to overlap other tiles' K loops: one slab of LDS and 128 registers, four workgroups per CU, rather
// than a deeper pipeline and two.  The accumulators meet the old statistics in registers - a half wavefront covers
// 128 consecutive bytes of a row, the mirror image is four consecutive floats per lane -, no pass through LDS.  In a
// whole tile they are read two pieces of 16 values ahead, and the fragments of a slab one step ahead: statistics of the 1.1B model,
// packed, 3.57 -> 3.43 ms; of one layer, full storage, 239 -> 231 us.  Two stages of 32 k with loads a slab ahead: 3.59 ms, 238 us.
// Up to two tiles per CU nothing overlaps a workgroup's waits but itself: two slabs of LDS then (ST = 2).  Us of a call, one / two: blocks of
// 1024 x 1024 (72 tiles) 1 20.5 / 19.4, 3 26.7 / 22.7, 5 33.2 / 30.8, 7 (504) 37.0 / 35.3, 9 (648) 47.8 / 52.0; packed 1000 x 2000 28.6 / 26.1.
constexpr int STATS_FEW_TILES = 512;
template <int ST>
__global__ __launch_bounds__(256, ST == 1 ? 4 : 2) void stats_product_kernel(const StatsEntry *__restrict__ entries, int count, int total,
                                                                             float beta)
{
    __shared__ __align__(16) unsigned char smem[32768 * ST];
    ASTERIA_LDS char *lds = (ASTERIA_LDS char *)smem;
    const int per_xcd = (total + NUM_XCD - 1) / NUM_XCD;
    const int t = (int)(blockIdx.x % NUM_XCD) * per_xcd + (int)(blockIdx.x / NUM_XCD);
    if (t >= total) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the entry of tile t: 64 candidates at a time
    int lo = 0, len = count;
    while (len > 1) {
        const int step = (len + 63) / 64, c = lo + lane * step;
        const bool le = lane * step < len && entries[c].tile_start <= t;
        const int last = 63 - __builtin_clzll(__ballot(le));
        lo += last * step;
        len = min(step, len - last * step);
    }
    lo = __builtin_amdgcn_readfirstlane(lo);
    const StatsEntry E = entries[lo];
    int lt = t - E.tile_start;
    const int tl = E.L ? tri_tiles(E.m) : 0;
    const bool left = lt < tl;
    if (!left) lt -= tl;
    int ti, tj;
    tri_decode(lt, ti, tj);
    const int n = left ? E.m : E.n, K = left ? E.n : E.m;
    const bool kmajor = !left && !(E.flags & STATS_TRANSPOSED), packed = (E.flags & STATS_PACKED) != 0;
    const int row0 = ti * 128, col0 = tj * 128;
    const bool diag = ti == tj;
    const int wm = wave >> 1, wn = wave & 1, r = lane & 31, h = lane >> 5;

    floatx16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    if (kmajor) stats_k_loop<true, ST>(acc, E.G, E.ldg, n, K, row0, col0, lds, wave, lane);
    else stats_k_loop<false, ST>(acc, E.G, E.ldg, n, K, row0, col0, lds, wave, lane);
    const int diag_d = diag ? wm - wn : 1;                    // < 0: above the diagonal
    if (diag_d < 0) return;

    // ---- old statistics in, new ones out
    const float alpha = 1.0f - beta;
    const int ldc = packed ? PACK_T : (left ? E.ldl : E.ldr);
    ASTERIA_GLOBAL float *C = (ASTERIA_GLOBAL float *)(left ? E.L : E.R);
    if (packed) C += ((size_t)ti * (ti + 1) / 2 + tj) * PACK_T * PACK_T - ((size_t)row0 * PACK_T + col0);   // of (0, 0) of the tile's frame
    const bool vec = (ldc & 3) == 0 && (reinterpret_cast<uintptr_t>(left ? E.L : E.R) & 15u) == 0;
    const bool read = beta != 0.0f;
    if (!diag && vec && read && ldc < (1 << 24) && row0 + 128 <= n && col0 + 128 <= n) {
        // a whole tile: pieces of 16 values of a lane (a block or its mirror image), the old values of the piece after next
        // on their way while one is combined and stored
        float o[2][16];
        int ln = lane;
        asm volatile("" : "+v"(ln));                          // addresses are made here, not kept through the K loop
        const uint32_t rr = (uint32_t)ln & 31u, hh = (uint32_t)ln >> 5;
        uint32_t lo4 = 16u * hh * (uint32_t)ldc + 4u * rr, lom = 4u * rr * (uint32_t)ldc + 16u * hh;     // bytes
        auto load = [&](float (&d)[16], int b, bool mirror) __attribute__((always_inline)) {
            const int br = row0 + (wm * 2 + (b >> 1)) * 32, bc = col0 + (wn * 2 + (b & 1)) * 32;
            if (!mirror) {
                const ASTERIA_GLOBAL float *cu = C + (size_t)br * ldc + bc;
#pragma unroll
                for (int v = 0; v < 16; ++v) d[v] = *(const ASTERIA_GLOBAL float *)((const ASTERIA_GLOBAL char *)(cu + (size_t)(8 * (v >> 2) + (v & 3)) * ldc) + lo4);
            } else {
                const ASTERIA_GLOBAL float *cu = C + (size_t)bc * ldc + br;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const floatx4 t = *(const ASTERIA_GLOBAL floatx4 *)((const ASTERIA_GLOBAL char *)(cu + 8 * g) + lom);
#pragma unroll
                    for (int e = 0; e < 4; ++e) d[4 * g + e] = t[e];
                }
            }
        };
        auto store = [&](const float (&d)[16], int b, bool mirror) __attribute__((always_inline)) {
            const int br = row0 + (wm * 2 + (b >> 1)) * 32, bc = col0 + (wn * 2 + (b & 1)) * 32;
            const floatx16 &p = acc[b >> 1][b & 1];
            if (!mirror) {
                ASTERIA_GLOBAL float *cu = C + (size_t)br * ldc + bc;
#pragma unroll
                for (int v = 0; v < 16; ++v) 
                    *(ASTERIA_GLOBAL float *)((ASTERIA_GLOBAL char *)(cu + (size_t)(8 * (v >> 2) + (v & 3)) * ldc) + lo4) = alpha * p[v] + beta * d[v];
            } else {
                ASTERIA_GLOBAL float *cu = C + (size_t)bc * ldc + br;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    floatx4 w;
#pragma unroll
                    for (int e = 0; e < 4; ++e) w[e] = alpha * p[4 * g + e] + beta * d[4 * g + e];
                    *(ASTERIA_GLOBAL floatx4 *)((ASTERIA_GLOBAL char *)(cu + 8 * g) + lom) = w;
                }
            }
        };
        auto all = [&](auto mirrors) __attribute__((always_inline)) {
            constexpr int U = decltype(mirrors)::value ? 8 : 4;
            load(o[0], 0, false);
            load(o[1], U == 8 ? 0 : 1, U == 8);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                __builtin_amdgcn_sched_barrier(0);
                asm volatile("" : "+v"(lo4), "+v"(lom));      // nor kept from one piece to the next
                store(o[u & 1], U == 8 ? u >> 1 : u, U == 8 && (u & 1));
                __builtin_amdgcn_sched_barrier(0);
                asm volatile("" : "+v"(lo4), "+v"(lom));
                if (u + 2 < U) load(o[u & 1], U == 8 ? (u + 2) >> 1 : u + 2, U == 8 && (u & 1));
            }
        };
        if (packed) all(std::false_type{}); else all(std::true_type{});
        return;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int br = row0 + (wm * 2 + i) * 32, bc = col0 + (wn * 2 + j) * 32;
            if (br < bc || br >= n || bc >= n) continue;      // blocks above the diagonal are mirror images
            const int col = bc + r;
            {
                ASTERIA_GLOBAL float *cu = C + (size_t)br * ldc + bc;         // uniform, beside a 32-bit lane offset
                const uint32_t lo4 = (uint32_t)(4 * h) * (uint32_t)ldc + (uint32_t)r;
                if (br + 32 <= n && bc + 32 <= n) {
                    float o[16];
                    if (read) {
#pragma unroll
                        for (int v = 0; v < 16; ++v) o[v] = (cu + (size_t)(8 * (v >> 2) + (v & 3)) * ldc)[lo4];
                    }
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const float p = alpha * acc[i][j][v];
                        (cu + (size_t)(8 * (v >> 2) + (v & 3)) * ldc)[lo4] = read ? p + beta * o[v] : p;
                    }
                } else {
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int row = br + 8 * (v >> 2) + 4 * h + (v & 3);
                        if (row < n && col < n) {
                            ASTERIA_GLOBAL float *cc = cu + (size_t)(8 * (v >> 2) + (v & 3)) * ldc + lo4;
                            const float p = alpha * acc[i][j][v];
                            *cc = read ? p + beta * *cc : p;
                        }
                    }
                }
            }
            // mirror image: a diagonal block holds both triangles itself (the products commute, so they agree bit for
            // bit); packed storage has none outside the diagonal tiles
            if (br == bc || (packed && !diag) || col >= n) continue;
            ASTERIA_GLOBAL float *c = C + (size_t)col * ldc + br + 4 * h;
            if (vec && br + 32 <= n) {
                floatx4 o[4];
                if (read) {
#pragma unroll
                    for (int g = 0; g < 4; ++g) o[g] = *(ASTERIA_GLOBAL floatx4 *)(c + 8 * g);
                }
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    floatx4 w;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float p = alpha * acc[i][j][4 * g + e];
                        w[e] = read ? p + beta * o[g][e] : p;
                    }
                    *(ASTERIA_GLOBAL floatx4 *)(c + 8 * g) = w;
                }
            } else {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int d = 8 * (v >> 2) + (v & 3);
                    if (br + 4 * h + d < n) {
                        const float p = alpha * acc[i][j][v];
                        c[d] = read ? p + beta * c[d] : p;
                    }
                }
            }
        }
}

}  // namespace asteria
