// Plane storage of square matrices and the pieces every kernel on it shares.
//
// A plane row holds, for every 32 consecutive k, NC segments of the same 32 values:
//   pair planes    NC = 2: value * scale = hi + lo as two fp16 terms, [32 hi][32 lo], 128 bytes - an fp32
//                  matrix kept to 22 bits in the bytes of an fp32 matrix
//   digit planes   NC = 4 or 5: value = integer * quantum, the integer of 8 NC bits as balanced
//                  base-256 digits (int8, most significant first), [32 d0][32 d1]..., 32 NC bytes
// Rows are padded with zeros to whole groups of 32 k.  The 16-byte chunks of a row piece are what one lane
// of an MFMA operand reads (8 fp16 or 16 int8 consecutive k of one row), so a product kernel moves operands
// from memory to LDS as they are: no conversion, no registers (buffer loads that write LDS directly).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gemm.h"

namespace asteria {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 pl_f16x8 __attribute__((ext_vector_type(8)));

__host__ __device__ inline int plane_groups(int n) { return (n + 31) / 32; }
__host__ __device__ inline int pair_row_bytes(int n) { return plane_groups(n) * 128; }
__host__ __device__ inline int digit_row_bytes(int n, int ns) { return plane_groups(n) * 32 * ns; }

// ---- global -> LDS ------------------------------------------------------------------------------
// Buffer descriptor over `bytes` bytes at p (wave-uniform).
__device__ __forceinline__ i32x4 buffer_rsrc(const void *p, uint32_t bytes)
{
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    i32x4 r;
    r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    r[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)((a >> 32) & 0xffffu));
    r[2] = __builtin_amdgcn_readfirstlane((int)bytes);
    r[3] = 0x00020000;
    return r;
}

// 16 bytes per lane from rsrc + voff + soff to LDS at lds_off + 16 * lane (lds_off, soff wave-uniform).
// The compiler does not see the load: wait_lds_loads counts it.  m0 is a reserved register, never allocated to a
// value, but the compiler writes it ahead of its own instructions that read it: the clobber keeps such a write from
// being shared across this statement (and earns a warning about reserved registers).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_to_lds(i32x4 rsrc, uint32_t lds_off, uint32_t voff, uint32_t soff)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(lds_off), "v"(voff), "s"(rsrc), "s"(soff) : "memory", "m0");
}
#pragma clang diagnostic pop

// All but the newest N vector-memory operations have arrived, and this wavefront's LDS reads are done
// (a slab may be overwritten once every wavefront has passed the barrier that follows).
template <int N> __device__ __forceinline__ void wait_lds_loads()
{
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "i"(N) : "memory");
}

// Operand rows of one workgroup tile: TMR rows of A and TNR rows of B, CPR 16-byte chunks per row piece,
// staged as they lie in memory except that chunk c of row r sits at position c ^ swz(r), so that the
// 16 rows that lanes read side by side fall into distinct 16-byte bank groups.  Rows beyond the matrix
// repeat its last row (their products are never stored).
template <int CPR> __device__ __forceinline__ int plane_swz(int r) { return CPR == 8 ? (r >> 1) & 7 : (r >> 3) & 1; }

template <int CPR, int TMR, int TNR, int NW>
struct PlaneLoader {
    static constexpr int CHUNKS = (TMR + TNR) * CPR;
    static constexpr int INSTR = CHUNKS / 64;                // load instructions per slab, NI per wavefront
    static constexpr int NI = (INSTR + NW - 1) / NW;
    static_assert(CHUNKS % 64 == 0 && (TMR * CPR) % 64 == 0, "whole instructions per operand");
    static constexpr int STAGE = CHUNKS * 16;
    i32x4 ra, rb;
    uint32_t vo[NI];
    int first;                                               // this wavefront's first instruction

    __device__ __forceinline__ void init(const char *A, const char *B, int rowb, int n, int row0, int col0, int wave, int lane)
    {
        ra = buffer_rsrc(A + (size_t)row0 * rowb, (uint32_t)TMR * (uint32_t)rowb);
        rb = buffer_rsrc(B + (size_t)col0 * rowb, (uint32_t)TNR * (uint32_t)rowb);
        first = wave * NI;
#pragma unroll
        for (int v = 0; v < NI; ++v) {
            const int p = min((first + v) * 64 + lane, CHUNKS - 1);   // chunk position within the stage
            const bool isb = (first + v) * 64 >= TMR * CPR;
            const int q = isb ? p - TMR * CPR : p;
            const int r = q / CPR, c = (q % CPR) ^ plane_swz<CPR>(r);
            const int lim = n - 1 - (isb ? col0 : row0);
            vo[v] = (uint32_t)min(r, lim) * (uint32_t)rowb + (uint32_t)c * 16u;
        }
    }
    __device__ __forceinline__ void issue(uint32_t lds_stage, int slab) const { issue_part(lds_stage, slab, 0, NI); }
    __device__ __forceinline__ void issue_part(uint32_t lds_stage, int slab, int v0, int v1) const     // instructions v0 .. v1 - 1 of NI
    {
#pragma unroll
        for (int v = v0; v < v1; ++v) {
            if (INSTR % NW != 0 && first + v >= INSTR) break;
            const bool isb = (first + v) * 64 >= TMR * CPR;
            load_to_lds(isb ? rb : ra, lds_stage + (uint32_t)(first + v) * 1024u, vo[v], (uint32_t)slab * (CPR * 16u));
        }
    }
};

// ---- elements <-> packed words --------------------------------------------------------------------
// A 32 x 32 accumulator block lies in lanes as: column r = lane % 32, rows 8 g + 4 h + e, h = lane / 32,
// register 4 g + e.  Its plane image needs consecutive columns of a row, its mirror image consecutive rows
// of a column; the latter is what a lane holds.

// 4 x 4 byte transpose: byte i of out[j] = byte j of in[i]
__device__ __forceinline__ void transpose4x4(const uint32_t (&w)[4], uint32_t (&o)[4])
{
    const uint32_t t0 = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u), t1 = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u);
    const uint32_t t2 = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u), t3 = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
    o[0] = __builtin_amdgcn_perm(t2, t0, 0x05040100u); o[1] = __builtin_amdgcn_perm(t2, t0, 0x07060302u);
    o[2] = __builtin_amdgcn_perm(t3, t1, 0x05040100u); o[3] = __builtin_amdgcn_perm(t3, t1, 0x07060302u);
}

// value (already scaled) -> hi | lo << 16, both terms rounded to nearest
__device__ __forceinline__ uint32_t pair_word(float v)
{
    const _Float16 h = (_Float16)v;
    const _Float16 l = (_Float16)(v - (float)h);
    return (uint32_t)__builtin_bit_cast(uint16_t, h) | ((uint32_t)__builtin_bit_cast(uint16_t, l) << 16);
}

// upper half of lanes of a <-> lower half of lanes of b
__device__ __forceinline__ void swap_halves(uint32_t &a, uint32_t &b)
{
    typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
    const u32x2_t r = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_permlane32_swap(a, b, false, false));
    a = r[0];
    b = r[1];
}

constexpr int PLANE_WORDS_PITCH = 36;                                     // 32 words + padding that keeps 16-byte alignment
constexpr int PLANE_SCRATCH_WORDS = 32 * PLANE_WORDS_PITCH;               // per wavefront
constexpr int PLANE_BYTES_PITCH = 48;
constexpr int PLANE_SCRATCH_BYTES = PLANE_SCRATCH_WORDS * 4 + 32 * PLANE_BYTES_PITCH;   // ... with a byte tile (5 digits)

// The block's words, one per element, turned so that lane (row = lane / 2, half = lane % 2) holds the 16
// words of columns 16 half .. of its row.  diag: the block lies on the diagonal of a symmetric matrix, its
// upper triangle is taken from the lower one.
__device__ __forceinline__ void words_by_row(ASTERIA_LDS uint32_t *ws, const uint32_t (&w)[16], int lane, bool diag, uint32_t (&x)[16])
{
    const int r = lane & 31, h = lane >> 5;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int v = 0; v < 16; ++v) ws[(8 * (v >> 2) + 4 * h + (v & 3)) * PLANE_WORDS_PITCH + r] = w[v];
    __builtin_amdgcn_wave_barrier();
    const int row = lane >> 1, c0 = (lane & 1) * 16;
    if (!diag) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const u32x4 t = *(const ASTERIA_LDS u32x4 *)(ws + row * PLANE_WORDS_PITCH + c0 + 4 * q);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[4 * q + e] = t[e];
        }
    } else {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int c = c0 + e;
            x[e] = ws[max(row, c) * PLANE_WORDS_PITCH + min(row, c)];
        }
    }
    __builtin_amdgcn_wave_barrier();
}

// Store a block of pair words at (br, bc) and, unless it lies on the diagonal, its mirror image.  Rows at or
// beyond n are not stored; the words of elements beyond n are zero (the padding of the rows).
__device__ __forceinline__ void store_pair_block(char *C, int rowb, int n, int br, int bc, const uint32_t (&w)[16], int lane,
                                                 ASTERIA_LDS uint32_t *ws)
{
    const bool diag = br == bc;
    {
        uint32_t x[16];
        words_by_row(ws, w, lane, diag, x);
        const int row = br + (lane >> 1);
        if (row < n) {
            char *p = C + (size_t)row * rowb + (bc >> 5) * 128 + (lane & 1) * 32;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                u32x4 hi, lo;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    hi[e] = __builtin_amdgcn_perm(x[8 * q + 2 * e + 1], x[8 * q + 2 * e], 0x05040100u);
                    lo[e] = __builtin_amdgcn_perm(x[8 * q + 2 * e + 1], x[8 * q + 2 * e], 0x07060302u);
                }
                *(ASTERIA_GLOBAL u32x4 *)(p + q * 16) = hi;
                *(ASTERIA_GLOBAL u32x4 *)(p + 64 + q * 16) = lo;
            }
        }
    }
    if (diag) return;
    uint32_t hw[4][2], lw[4][2];
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            hw[g][q] = __builtin_amdgcn_perm(w[4 * g + 2 * q + 1], w[4 * g + 2 * q], 0x05040100u);
            lw[g][q] = __builtin_amdgcn_perm(w[4 * g + 2 * q + 1], w[4 * g + 2 * q], 0x07060302u);
        }
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int q = 0; q < 2; ++q) { swap_halves(hw[g][q], hw[g + 2][q]); swap_halves(lw[g][q], lw[g + 2][q]); }
    // lanes of the lower half now hold rows 0 .. 15 of their column, the upper half rows 16 .. 31
    const int col = bc + (lane & 31), h = lane >> 5;
    if (col < n) {
        char *p = C + (size_t)col * rowb + (br >> 5) * 128 + h * 32;
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            *(ASTERIA_GLOBAL u32x4 *)(p + g * 16) = (u32x4){hw[g][0], hw[g][1], hw[g + 2][0], hw[g + 2][1]};
            *(ASTERIA_GLOBAL u32x4 *)(p + 64 + g * 16) = (u32x4){lw[g][0], lw[g][1], lw[g + 2][0], lw[g + 2][1]};
        }
    }
}

// ---- digits ----------------------------------------------------------------------------------------
// Balanced base-256 digits of an integer: adding 128 at every lower digit and flipping the top bit of the
// bytes turns two's complement into digits in [-128, 127].  NS = 4: |v| <= 0x7f7f7f7f; NS = 5: the low
// word holds digits 1 .. 4, the top digit comes back in `top`.
constexpr double DIGIT_LIMIT4 = 2139062143.0;                 // 0x7f7f7f7f
constexpr double DIGIT_LIMIT5 = 2139062143.0 * 256.0 + 127.0;
__device__ __forceinline__ int undigits4(uint32_t w) { return (int)((w ^ 0x00808080u) - 0x00808080u); }

// x rounded to an integer in the digit range -> low word (and top digit); values beyond the range saturate and set `over`.
// The rounding is that of an addition to 2^52 + 2^51, whose last bit is worth 1: the integer, already in the balanced form's offset,
// is then the lower part of the sum's mantissa, without a conversion.
template <int NS>
__device__ __forceinline__ uint32_t digit_word(double x, uint32_t &top, bool &over)
{
    constexpr double lim = NS == 4 ? DIGIT_LIMIT4 : DIGIT_LIMIT5;
    constexpr uint32_t offset = NS == 4 ? 0x00808080u : 0x80808080u;
    if (!(fabs(x) < lim + 0.5)) { over = true; x = x > 0.0 ? lim : (x < 0.0 ? -lim : 0.0); }
    const uint64_t t = (uint64_t)__double_as_longlong(x + (6755399441055744.0 + (double)offset));
    top = NS == 4 ? 0u : (uint32_t)(t >> 32) & 0xffu;
    return (uint32_t)t ^ offset;
}

// 16 words of 16 consecutive k of one row -> one 16-byte chunk per digit, digit s at p + 32 s
template <int NS>
__device__ __forceinline__ void store_digit_chunk(char *p, const uint32_t (&x)[16], u32x4 top)
{
    uint32_t d[4][4];                                          // [digit from the least significant][4 k]
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t in[4] = {x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]};
        uint32_t o[4];
        transpose4x4(in, o);
#pragma unroll
        for (int s = 0; s < 4; ++s) d[s][q] = o[s];
    }
    if constexpr (NS == 5) *(ASTERIA_GLOBAL u32x4 *)p = top;
#pragma unroll
    for (int s = 0; s < 4; ++s)
        *(ASTERIA_GLOBAL u32x4 *)(p + 32 * (NS - 1 - s)) = (u32x4){d[s][0], d[s][1], d[s][2], d[s][3]};
}

// Store a block of digit words (w: low words, tp: top digits, four registers' to a word) at (br, bc) and its mirror image.
template <int NS>
__device__ __forceinline__ void store_digit_block(char *C, int rowb, int n, int br, int bc, const uint32_t (&w)[16],
                                                  const uint32_t (&tp)[4], int lane, ASTERIA_LDS uint32_t *ws)
{
    const bool diag = br == bc;
    const int r = lane & 31, h = lane >> 5;
    {
        uint32_t x[16];
        u32x4 top = {0u, 0u, 0u, 0u};
        if constexpr (NS == 5) {
            ASTERIA_LDS uint8_t *bs = (ASTERIA_LDS uint8_t *)(ws + PLANE_SCRATCH_WORDS);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = 8 * (v >> 2) + 4 * h + (v & 3);
                bs[row * PLANE_BYTES_PITCH + r] = (uint8_t)(tp[v >> 2] >> (8 * (v & 3)));
            }
            __builtin_amdgcn_wave_barrier();
            const int row = lane >> 1, c0 = (lane & 1) * 16;
            if (!diag) {
                top = *(const ASTERIA_LDS u32x4 *)(bs + row * PLANE_BYTES_PITCH + c0);
            } else {
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int c = c0 + e;
                    top[e >> 2] |= (uint32_t)bs[max(row, c) * PLANE_BYTES_PITCH + min(row, c)] << (8 * (e & 3));
                }
            }
        }
        words_by_row(ws, w, lane, diag, x);
        const int row = br + (lane >> 1);
        if (row < n) store_digit_chunk<NS>(C + (size_t)row * rowb + (bc >> 5) * (32 * NS) + (lane & 1) * 16, x, top);
    }
    if (diag) return;
    uint32_t d[NS][4];                                         // [digit, most significant first][g]: 4 rows of the lane's column
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const uint32_t in[4] = {w[4 * g], w[4 * g + 1], w[4 * g + 2], w[4 * g + 3]};
        uint32_t o[4];
        transpose4x4(in, o);
#pragma unroll
        for (int s = 0; s < 4; ++s) d[NS - 1 - s][g] = o[s];
        if constexpr (NS == 5) d[0][g] = tp[g];
    }
    const int col = bc + r;
    char *p = C + (size_t)col * rowb + (br >> 5) * (32 * NS) + h * 16;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        swap_halves(d[s][0], d[s][2]);
        swap_halves(d[s][1], d[s][3]);
        if (col < n) *(ASTERIA_GLOBAL u32x4 *)(p + 32 * s) = (u32x4){d[s][0], d[s][2], d[s][1], d[s][3]};
    }
}

// The block of a symmetric digit plane at (br, bc) in accumulator order (integers as doubles), from its mirror image: groups q and
// q + 2 of four rows (q = 0 or 1).  p: digit 0 of rows br + 16 h .. of the lane's column, h = lane / 32.  A half wavefront reads 8 bytes
// of the 16 and trades those the other half needs.
template <int NS>
__device__ __forceinline__ void load_digit_groups(const char *p, int q, double (&v)[2][4])
{
    typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
    uint32_t b[2][NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const u32x2_t w = *(const ASTERIA_GLOBAL u32x2_t *)(p + 32 * s + 8 * q);
        b[0][s] = w[0]; b[1][s] = w[1];
        swap_halves(b[0][s], b[1][s]);
    }
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        const uint32_t in[4] = {b[g][NS - 1], b[g][NS - 2], b[g][NS - 3], b[g][NS - 4]};
        uint32_t o[4];
        transpose4x4(in, o);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if constexpr (NS == 4) v[g][e] = (double)undigits4(o[e]);
            else {
                // low word: four balanced digits, sum in [-0x80808080, 0x7f7f7f7f]
                const int t = (int)(b[g][0] << (24 - 8 * e)) >> 24;
                v[g][e] = fma((double)t, 4294967296.0, (double)(o[e] ^ 0x80808080u)) - 2155905152.0;
            }
        }
    }
}

}  // namespace asteria
