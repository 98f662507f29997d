// Launch interface of the wide products with packed input rows (dense_kernels.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "cell_kernels.h"

namespace acrobat {

// Where the states of tree nodes go besides the arena: the operands of the blocks that read them (packed_kernels.hip).
struct TreePlaces {
  void* operand; uint32_t operand_bytes;  // null: nowhere
  float* cells;
  const int32_t* place;  // [n] by list position
};

constexpr int32_t kDenseMaxK = 1024;
constexpr double kDenseMaxBytes = 4294967296.0 - 131072.0;

// Input rows as matrix operands: blocks of 16 rows, 64 K bytes each, every row's inverse scale and the largest of a block.
struct PackRowsArgs {
  int32_t n, K;
  const float* src; const int32_t* idx;  // row of src by position, null: the position itself
  void* operand;   // [ceil(n / 16)] blocks
  float* inverse;  // [16 ceil(n / 16)]
  float* largest;  // [ceil(n / 16)]
};

// One level: TREE_LEAF, STORE_Z or STORE_Z1 with one segment of at most kDenseMaxK columns, H a multiple of 32; `two`: odd
// groups work with b, another batch of the same sizes over the same input rows.
struct DenseArgs {
  CellLevelArgs a, b;
  int32_t two;
  const void* operand; uint32_t operand_bytes;
  float* inverse;
  const float* largest;
  TreePlaces places;
  int32_t n_cb, n_groups;  // set by the launcher
};
// Whether a level (G gates of H units over K columns) is wide enough for this kernel to win; a forced tile switches it off.
bool dense_level_wins(CellEpilogue epi, int32_t n, int32_t H, int32_t K, const SplitKWorkspace& ws);
// Scratch of a level: packed rows, then their inverse scales, then the largest ones; whole cache lines, so that what lies
// behind it is aligned.
inline size_t dense_scratch_bytes(int32_t n, int32_t K) {
  const size_t blocks = ((size_t)n + 15) / 16;
  return blocks * (16 * (size_t)K + 32) * sizeof(float);
}
// Packs the input rows (s.a.src0, gathered by s.a.idx0) into `scratch` and runs the level: two launches.  A leaf level (its rows
// and its results are named by lists) runs in pieces, with the same bits, where not all of its rows fit.
hipError_t launch_dense_level(CellEpilogue epi, const DenseArgs& s, void* scratch, size_t scratch_bytes, int n_cu,
                              hipStream_t stream, const LaunchEvents& ev = LaunchEvents());

}  // namespace acrobat
