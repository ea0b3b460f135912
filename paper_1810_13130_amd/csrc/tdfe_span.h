// Where the lanes of a block operator kernel read: plain integer arithmetic
// without HIP, so that the host can go through every lane of a launch.
#pragma once
#include <cstdint>

#ifdef __HIPCC__
#define TDFE_HD __host__ __device__ __forceinline__
#else
#define TDFE_HD inline
#endif

namespace tdfe_span {

// a byte offset past the end of every buffer resource of these kernels (they
// hold at most 2^31 - 1 bytes): the load gives 0 and touches no memory
constexpr uint32_t NO_READ = 0x80000000u;

// Byte offset of a lane's node (0, j, 0) of a trilinear cell from the start of
// the block's buffer resource, `rows` DoF rows on; its other nodes add (row
// difference) ld size bytes, less than 2^31.  The resource ends with the last
// row's ld columns counted from its start, and a launch on columns col0.. of a
// wider vector starts col0 columns into a row: what lies past such a launch's
// own columns in the last row is past the vector, so lanes without a column
// (the last column block's padding) or without a cell must not read.
TDFE_HD int64_t gather_offset(bool act, int64_t rows, int ld, int colg, int size) {
  return act ? (rows * ld + colg) * size : (int64_t)NO_READ;
}

}  // namespace tdfe_span
