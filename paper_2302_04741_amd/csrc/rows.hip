// Population import and export: dense rows <-> the padded rows of the planes.
#include <algorithm>

#include "lbm_internal.h"

namespace lbm {

namespace {
typedef uint32_t Words4 __attribute__((ext_vector_type(4)));
// the same 16 bytes at the alignment of one element
template <class E> struct LooseVec;
template <> struct LooseVec<uint64_t> {
    typedef uint32_t type __attribute__((ext_vector_type(4), aligned(8)));
};
template <> struct LooseVec<uint32_t> {
    typedef uint32_t type __attribute__((ext_vector_type(4), aligned(4)));
};
template <> struct LooseVec<uint16_t> {
    typedef uint32_t type __attribute__((ext_vector_type(4), aligned(2)));
};

struct RowCopy {
    char *padded;    // rows of `pitch` bytes
    char *dense;     // n elements, back to back
    uint64_t pitch;
    uint64_t n;
    uint64_t chunks; // whole 16-byte chunks of the dense side
    uint32_t nx;     // elements a row
    uint32_t head;   // elements before the dense side's first 16-byte boundary
    DivU32 by_nx;
};

constexpr int CHUNKS = 8;                    // 16-byte chunks a thread
constexpr uint32_t BLOCK_CHUNKS = 256 * CHUNKS;

// 16 bytes a lane on 16-byte boundaries of the dense side, 32 KB a block; a chunk's
// place in the padded rows comes from one division by nx, and a chunk that runs
// over a row's end takes the padded side element by element.  Bound by memory: it
// reads and writes the state once.  us of an export, against the runtime's 2-D
// copy: D2Q37 1017^2 FP32 49 / 108, D3Q39 121x99x141 F16 50 / 269, 129x95x110 FP64
// 166 / 293, 10x302x138 FP64 69 / 71.  (A wavefront a row did as well on long rows
// and took up to three times the runtime's time on rows of 10 to 60 values.)
template <class E, bool EXPORT>
__global__ void __launch_bounds__(256) copy_rows_kernel(RowCopy c)
{
    using Loose = typename LooseVec<E>::type;
    constexpr uint32_t EPC = 16 / sizeof(E);
    const uint64_t first = uint64_t(blockIdx.x) * BLOCK_CHUNKS;
    // the block's first element: its row and place in it (uniform)
    const uint64_t e0 = c.head + first * EPC;
    const uint64_t r0 = e0 / c.nx;
    const uint32_t x0 = uint32_t(e0 - r0 * c.nx);
    char *dense = c.dense + e0 * sizeof(E);
    Words4 v[CHUNKS];
    char *at[CHUNKS];
    uint32_t left[CHUNKS];  // elements to the end of the row
#pragma unroll
    for (int k = 0; k < CHUNKS; ++k) {
        const uint32_t j = uint32_t(k) * 256u + threadIdx.x;
        const uint32_t e = x0 + j * EPC;  // < nx + 2^14, nx <= 2^30
        const uint32_t r = divu(c.by_nx, e);
        const uint32_t x = e - r * c.nx;
        left[k] = c.nx - x;
        at[k] = c.padded + (r0 + r) * c.pitch + uint64_t(x) * sizeof(E);
        if (first + j >= c.chunks) continue;
        if (!EXPORT) {
            v[k] = *reinterpret_cast<const Words4 *>(dense + uint64_t(j) * 16);
        } else if (left[k] >= EPC) {
            v[k] = *reinterpret_cast<const Loose *>(at[k]);
        } else {
            E w[EPC];
            const char *p = at[k];
            uint32_t l = left[k];
#pragma unroll
            for (uint32_t q = 0; q < EPC; ++q) {
                w[q] = *reinterpret_cast<const E *>(p);
                p += sizeof(E);
                if (--l == 0) {
                    p += c.pitch - uint64_t(c.nx) * sizeof(E);
                    l = c.nx;
                }
            }
            __builtin_memcpy(&v[k], w, 16);
        }
    }
#pragma unroll
    for (int k = 0; k < CHUNKS; ++k) {
        const uint32_t j = uint32_t(k) * 256u + threadIdx.x;
        if (first + j >= c.chunks) continue;
        if (EXPORT) {
            *reinterpret_cast<Words4 *>(dense + uint64_t(j) * 16) = v[k];
        } else if (left[k] >= EPC) {
            *reinterpret_cast<Loose *>(at[k]) = v[k];
        } else {
            E w[EPC];
            __builtin_memcpy(w, &v[k], 16);
            char *p = at[k];
            uint32_t l = left[k];
#pragma unroll
            for (uint32_t q = 0; q < EPC; ++q) {
                *reinterpret_cast<E *>(p) = w[q];
                p += sizeof(E);
                if (--l == 0) {
                    p += c.pitch - uint64_t(c.nx) * sizeof(E);
                    l = c.nx;
                }
            }
        }
    }
    // the elements before the first and after the last whole chunk, at most 7 each
    if (blockIdx.x == 0 && threadIdx.x < 16) {
        const uint64_t tail = c.head + c.chunks * EPC;  // first element after the chunks
        const uint64_t e = threadIdx.x < 8 ? threadIdx.x : tail + (threadIdx.x - 8);
        if (threadIdx.x < 8 ? e < c.head : e < c.n) {
            const uint64_t r = e / c.nx;
            E *p = reinterpret_cast<E *>(c.padded + r * c.pitch) + (e - r * c.nx);
            E *d = reinterpret_cast<E *>(c.dense) + e;
            if (EXPORT) *d = *p;
            else *p = *d;
        }
    }
}

template <class E> void launch_rows(const RowCopy &c, bool exporting, hipStream_t stream)
{
    const unsigned blocks =
        unsigned(std::max<uint64_t>(1, (c.chunks + BLOCK_CHUNKS - 1) / BLOCK_CHUNKS));
    if (exporting)
        hipLaunchKernelGGL((copy_rows_kernel<E, true>), dim3(blocks), dim3(256), 0, stream, c);
    else
        hipLaunchKernelGGL((copy_rows_kernel<E, false>), dim3(blocks), dim3(256), 0, stream, c);
}
}  // namespace

hipError_t launch_copy_rows(int storage, void *padded, void *dense, const GridDims &gd, int Q,
                            bool exporting, hipStream_t stream)
{
    const uint64_t sb = storage == 0 ? 8 : (storage == 1 ? 4 : 2);
    RowCopy c{};
    c.padded = static_cast<char *>(padded);
    c.dense = static_cast<char *>(dense);
    c.pitch = uint64_t(gd.px) * sb;
    c.n = uint64_t(Q) * uint64_t(gd.N);
    c.nx = uint32_t(gd.nx);
    c.by_nx = make_divu32(c.nx);
    const uint64_t off = (16 - reinterpret_cast<uintptr_t>(dense) % 16) % 16 / sb;
    c.head = uint32_t(std::min<uint64_t>(off, c.n));
    c.chunks = (c.n - c.head) * sb / 16;
    if (storage == 0) launch_rows<uint64_t>(c, exporting, stream);
    else if (storage == 1) launch_rows<uint32_t>(c, exporting, stream);
    else launch_rows<uint16_t>(c, exporting, stream);
    return hipGetLastError();
}

}  // namespace lbm
