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
    char *padded;      // rows of `pitch` bytes, 128-byte aligned
    char *dense;       // rows of `row` bytes, back to back
    uint64_t pitch, row;
    uint32_t tasks;    // rows x pieces of a row
    uint32_t pieces;
    DivU32 by_pieces;
};

constexpr int CHUNKS = 8;                            // 16-byte chunks a lane and task
constexpr uint64_t PIECE = uint64_t(CHUNKS) * 64;    // chunks a task

// One wavefront copies a piece of one row (8 KB): 16 bytes a lane on 16-byte
// boundaries of the dense side, whose rows start anywhere, so the padded side is
// accessed at the element's alignment; the elements before the first and after
// the last boundary go one a lane.  Bound by memory: it reads and writes the state
// once.  D2Q37 1017^2 FP32 (307 MB both ways): hipMemcpy2DAsync 104-110 us.
template <class E, bool EXPORT>
__global__ void __launch_bounds__(256) copy_rows_kernel(RowCopy c)
{
    using Loose = typename LooseVec<E>::type;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t waves = gridDim.x * 4u;
    for (uint32_t t = __builtin_amdgcn_readfirstlane(blockIdx.x * 4u + (threadIdx.x >> 6));
         t < c.tasks; t += waves) {
        const uint32_t r = divu(c.by_pieces, t);
        const uint32_t piece = t - r * c.pieces;
        char *d = c.dense + uint64_t(r) * c.row;
        char *p = c.padded + uint64_t(r) * c.pitch;
        uint64_t head = (16u - (reinterpret_cast<uint64_t>(d) & 15u)) & 15u;
        head = head < c.row ? head : c.row;
        const uint64_t body = (c.row - head) / 16;  // whole chunks
        const uint32_t tail = uint32_t(c.row - head - body * 16);
        Words4 v[CHUNKS];
#pragma unroll
        for (int k = 0; k < CHUNKS; ++k) {
            const uint64_t at = piece * PIECE + uint32_t(k) * 64u + lane;
            if (at < body)
                v[k] = EXPORT ? Words4(*reinterpret_cast<const Loose *>(p + head + at * 16))
                              : *reinterpret_cast<const Words4 *>(d + head + at * 16);
        }
        // elements outside the chunks: the head's in lanes 0-7, the tail's in 8-15
        const uint32_t nh = piece == 0 ? uint32_t(head / sizeof(E)) : 0u;
        const uint32_t nt = piece + 1 == c.pieces ? uint32_t(tail / sizeof(E)) : 0u;
        const bool edge = lane < 8u ? lane < nh : lane - 8u < nt;
        const uint64_t off = (lane < 8u ? lane * sizeof(E)
                                        : c.row - tail + (lane - 8u) * sizeof(E));
        if (edge) {
            if (EXPORT) *reinterpret_cast<E *>(d + off) = *reinterpret_cast<const E *>(p + off);
            else *reinterpret_cast<E *>(p + off) = *reinterpret_cast<const E *>(d + off);
        }
#pragma unroll
        for (int k = 0; k < CHUNKS; ++k) {
            const uint64_t at = piece * PIECE + uint32_t(k) * 64u + lane;
            if (at < body) {
                if (EXPORT) *reinterpret_cast<Words4 *>(d + head + at * 16) = v[k];
                else *reinterpret_cast<Loose *>(p + head + at * 16) = Loose(v[k]);
            }
        }
    }
}

template <class E>
void launch_rows(const RowCopy &c, bool exporting, hipStream_t stream)
{
    const unsigned blocks = unsigned(std::min<uint64_t>((uint64_t(c.tasks) + 3) / 4, 1u << 20));
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
    c.row = uint64_t(gd.nx) * sb;
    c.pieces = uint32_t(std::max<uint64_t>(1, (c.row / 16 + PIECE - 1) / PIECE));
    c.by_pieces = make_divu32(c.pieces);
    // a plane is < 4 GiB, so all rows (at least 128 bytes) and pieces stay below 2^32
    c.tasks = uint32_t(uint64_t(Q) * uint64_t(gd.ny) * uint64_t(gd.nz) * c.pieces);
    if (storage == 0) launch_rows<uint64_t>(c, exporting, stream);
    else if (storage == 1) launch_rows<uint32_t>(c, exporting, stream);
    else launch_rows<uint16_t>(c, exporting, stream);
    return hipGetLastError();
}

}  // namespace lbm
