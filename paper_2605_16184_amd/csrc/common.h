// Host-side helpers shared by the entry points: argument checks, workspace carving and the
// asynchronous host -> device table upload.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>

#include "../../include/asteria.h"

namespace asteria {

#define ASTERIA_HIP_TRY(expr)                          \
    do {                                               \
        hipError_t e__ = (expr);                       \
        if (e__ != hipSuccess) return ASTERIA_HIP_ERROR; \
    } while (0)

#define ASTERIA_TRY(expr)                              \
    do {                                               \
        asteria_status s__ = (expr);                   \
        if (s__ != ASTERIA_OK) return s__;             \
    } while (0)

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Sequential carving of a caller-owned workspace into 256-byte aligned pieces.
struct Carver {
    unsigned char *base;
    size_t off;
    explicit Carver(void *p) : base(reinterpret_cast<unsigned char *>(p)), off(0) {}
    template <typename T> T *take(size_t count)
    {
        T *p = reinterpret_cast<T *>(base + off);
        off += align_up(count * sizeof(T), 256);
        return p;
    }
    static size_t need(size_t count, size_t elem) { return align_up(count * elem, 256); }
};

// Host -> device copies that are ordered on the stream, never block and never read host memory after they
// return: the bytes travel as by-value kernel arguments, one chunk per launch.  A launch is 4.5 us in a chain however little
// it carries, so the tables of a call share chunks: add() takes the bytes, flush() launches what add() has not.
// SOAP period boundary of 9 blocks: 11 launches of the step and the reprojection before, 4 now.
constexpr int UPLOAD_WORDS = 896, UPLOAD_PIECES = 8;   // below the 4 KiB argument limit; whole 16-byte pieces
struct alignas(16) UploadChunk {
    uint32_t w[UPLOAD_WORDS];
    uint32_t *dst[UPLOAD_PIECES];
    int begin[UPLOAD_PIECES], end[UPLOAD_PIECES];      // of the piece within w; begin a multiple of 4
};
static_assert(sizeof(UploadChunk) <= 3840, "argument limit");

// Kernel arguments lie in host memory: every lane makes one load.
static __global__ __launch_bounds__(256) void upload_chunk_kernel(UploadChunk chunk, int pieces)
{
    typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
    const int i = (int)threadIdx.x * 4;
    if (i >= UPLOAD_WORDS) return;
    const u32x4_t v = *reinterpret_cast<const u32x4_t *>(chunk.w + i);
    for (int p = 0; p < pieces; ++p) {
        const int b = chunk.begin[p], n = chunk.end[p];
        if (i < b || i >= n) continue;
        uint32_t *d = chunk.dst[p] + (i - b);
#pragma unroll
        for (int e = 0; e < 4; ++e) if (i + e < n) d[e] = v[e];
    }
}

class Uploads {
public:
    explicit Uploads(hipStream_t stream) : stream_(stream) {}
    // dst must be 4-byte aligned; bytes is rounded up to whole words (dst needs that much room)
    hipError_t add(void *dst, const void *src, size_t bytes)
    {
        const unsigned char *s = reinterpret_cast<const unsigned char *>(src);
        uint32_t *d = reinterpret_cast<uint32_t *>(dst);
        while (bytes > 0) {
            if (words_ == UPLOAD_WORDS || pieces_ == UPLOAD_PIECES)
                if (hipError_t e = flush(); e != hipSuccess) return e;
            const size_t room = (size_t)(UPLOAD_WORDS - words_) * 4, take = bytes < room ? bytes : room;
            const int nwords = (int)((take + 3) / 4);
            chunk_.w[words_ + nwords - 1] = 0;
            memcpy(chunk_.w + words_, s, take);
            chunk_.dst[pieces_] = d;
            chunk_.begin[pieces_] = words_;
            chunk_.end[pieces_] = words_ + nwords;
            ++pieces_;
            words_ += (nwords + 3) / 4 * 4;
            s += take; d += nwords; bytes -= take;
        }
        return hipSuccess;
    }
    hipError_t flush()
    {
        if (pieces_ == 0) return hipSuccess;
        hipLaunchKernelGGL(upload_chunk_kernel, dim3(1), dim3(256), 0, stream_, chunk_, pieces_);
        pieces_ = words_ = 0;
        return hipGetLastError();
    }

private:
    hipStream_t stream_;
    UploadChunk chunk_ = {};
    int words_ = 0, pieces_ = 0;
};

inline hipError_t upload_async(void *dst, const void *src, size_t bytes, hipStream_t stream)
{
    Uploads u(stream);
    if (hipError_t e = u.add(dst, src, bytes); e != hipSuccess) return e;
    return u.flush();
}

inline bool valid_dtype(int d) { return d == ASTERIA_F32 || d == ASTERIA_BF16; }

}  // namespace asteria
