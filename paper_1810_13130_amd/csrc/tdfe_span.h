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

// DoF rows from node (0, 0, 0) of the first to the last node of the last of
// `cells` consecutive cells, the most over all positions of the first on a
// grid of ncx x ncy x ncz cells of order p
inline int64_t block_rows(int p, int64_t ncx, int64_t ncy, int64_t ncz, int64_t cells) {
  const int64_t row = ncx * p - 1, layer = row * (ncy * p - 1), per = ncx * ncy;
  int64_t most = 0;
  for (int64_t d = 0; d < cells && d < per * ncz; ++d)
    for (int64_t dz = d / per; dz <= d / per + 1 && dz < ncz; ++dz) {
      const int64_t e = d - dz * per;  // y and x differences of cells d apart, dz layers apart
      const int64_t y0 = e >= 0 ? e / ncx : -((-e + ncx - 1) / ncx);
      for (int64_t dy = y0; dy <= y0 + 1; ++dy) {
        const int64_t dx = e - dy * ncx;
        if (dy <= -ncy || dy >= ncy || dx <= -ncx || dx >= ncx) continue;
        const int64_t r = p * (dz * layer + dy * row + dx);
        if (r > most) most = r;
      }
    }
  return most + p * (layer + row + 1);
}

// whether 32-bit byte offsets reach every node of a block of that many cells
// (one row further for the columns within a row)
inline bool near(int p, int64_t ncx, int64_t ncy, int64_t ncz, int64_t cells, int64_t row_bytes) {
  return (block_rows(p, ncx, ncy, ncz, cells) + 1) * row_bytes < (int64_t)1 << 31;
}

}  // namespace tdfe_span
