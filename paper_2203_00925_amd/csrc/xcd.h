// Block order for gather kernels on the 8 XCDs of the chip.  Blocks are
// dealt to the XCDs in turn and each XCD has its own L2; with the grid
// padded to a multiple of 8, block b works on logical block
// (b % 8) * (grid / 8) + b / 8, so each XCD takes one contiguous eighth of
// the rows and the neighbour data that consecutive rows share (nearby cells
// of a space-filling-curve order) stays in one L2.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace mifvm {

constexpr int kXcds = 8;

__device__ inline int64_t xcd_block() {
    const int64_t per = gridDim.x / kXcds;
    return int64_t(blockIdx.x % kXcds) * per + blockIdx.x / kXcds;
}
__device__ inline int64_t gtid_m() { return xcd_block() * blockDim.x + threadIdx.x; }
// a grid of n blocks padded to a multiple of 8; one of blocks of `block` threads covering n rows
inline unsigned pad8(int64_t n) { return unsigned((n + kXcds - 1) / kXcds * kXcds); }
inline unsigned rows_m(int64_t n, int block) { return pad8((n + block - 1) / block); }

// The same for a step's kernels, which read some dozen arrays once: above
// 4,096 blocks (1M cells, or 262k vertices of the moments) the XCDs take
// windows of 32 blocks each in turn.  Eight distant streams per array cost the
// HBM a tenth of its rate (eleven arrays of 3.1M 16-byte items: 5.31 TB/s in
// eighths, 5.88 in plain order), and a window of 8,192 rows keeps nearly all of
// their neighbours in its L2.  Measured on both sides of the line, not at it:
// two steps at 3.07M cells (12,000 blocks) eighths 2,067 us, windows of 8
// blocks 2,015, of 32 2,011, of 128 2,050; four at 304k (1,187 blocks) eighths
// 478, windows of 32 498.
// The order is an argument: a choice between the two in the kernel is a branch
// before its first load (48k cells, ten steps: 459 us against 442).
struct BlockOrder {
    unsigned grid;                        // blocks to launch
    unsigned shift, width;                // a round is 8 windows of `width` = 2^shift blocks, or one of eighths
    __device__ int64_t block() const {
        const unsigned q = blockIdx.x / kXcds, x = blockIdx.x % kXcds;
        return (q >> shift << (shift + 3)) + x * width + (q & ((1u << shift) - 1u));
    }
};
inline BlockOrder stream_order(int64_t rows, int rows_per_block) {
    const int64_t n = (rows + rows_per_block - 1) / rows_per_block;
    constexpr unsigned W = 32;
    if (n > 4096) return {unsigned((n + kXcds * W - 1) / (kXcds * W) * (kXcds * W)), 5u, W};
    const unsigned g = pad8(n);
    return {g, 28u, g / kXcds};
}

}  // namespace mifvm
