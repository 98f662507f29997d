// Launch interface of the weight-stationary cell kernels (tree_kernels.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "cell_kernels.h"

namespace acrobat {

constexpr int kTreeMaxGroups = 256;
constexpr int kTreeCounterStride = 32;  // uint32 between two groups' arrival counters (a cache line each)
constexpr int kStationaryMaxK = 1024;   // columns of the contraction that fit the register files
constexpr int kStationaryMaxStepK = 512;  // the same for the steps of a recurrence

// Rows [list positions] of one or more levels.  a: the batch as for a level launch, with idx0 / idx1 / out_rows indexed
// by absolute list position (null: the position itself) and, if off is null, n rows; both segments of a TREE_INTERNAL
// contraction are rows of src0.  LSTM_STEP and RNN_STEP (packed_kernels.hip) read the row of src0 before the one they write,
// the odd groups of two directions the one behind it.
struct StationaryArgs {
  CellLevelArgs a[2];
  int32_t two;             // != 0: odd groups work with a[1] (the two directions of a bidirectional recurrence)
  uint32_t src_bytes;      // of src0, at most 2^32 - 512
  int32_t n_cb;            // workgroups of a group: H / 16, of packed recurrences packed_members
  int32_t n_groups;
  // off[lv * n_groups + g]: first list position of group g's share of level lv; levels follow one another, so the entry
  // behind it is the end of the share.  null: one level of a.n rows, shared evenly.
  const int32_t* off;
  int32_t level0, level1;  // levels to run; with more than one the workgroups of a group wait for each other
  unsigned* counters;      // [n_groups * kTreeCounterStride], zero at launch and again when the launch has completed
  unsigned* status;
  int32_t max_polls;
  unsigned long long* stamps;  // [levels * n_groups] 100 MHz clock at the end of a group's share of a level, or null
  // packed_kernels.hip, and the operands that leaves go to: the operands of all blocks, split states and c states, and every
  // list position's place in them, 2 (16 block + row of the node that reads it) + side; -1: nobody reads it here
  void* operand; uint32_t operand_bytes;  // at most kPackedMaxBytes
  float* cells;
  const int32_t* place;    // trees only
  int32_t n_steps;         // of a recurrence, also those behind level1
  int32_t first_position;  // trees: list position from which blocks are counted
  int32_t share_blocks;    // recurrences: blocks of a group's share of any step but the first
  int32_t sets;            // and sets of blocks that the steps take in turn
  int32_t variant;         // which instance, see packed_variant
};
// Groups of H / 16 workgroups that are resident on the current device at once (eight XCDs, a group never crosses one);
// 0 if the contraction does not fit.
int stationary_groups(CellEpilogue epi, int32_t H, int32_t K, int32_t n_cu);
hipError_t launch_stationary(CellEpilogue epi, const StationaryArgs& s, hipStream_t stream, const LaunchEvents& ev = LaunchEvents());
// One internal level [level0, level0 + 1) of trees, list positions [p_first, p_first + n), by a launch that waits for
// nothing: the same kernel, or for levels of a few blocks one in which several workgroups share a block's contraction
// (partial sums and tickets in ws, tickets zero before and after).  The same results either way.
constexpr int32_t kPartsMaxRows = 64;
hipError_t launch_tree_level(const StationaryArgs& s, int32_t p_first, int32_t n, const SplitKWorkspace& ws, hipStream_t stream,
                             const LaunchEvents& ev = LaunchEvents());

// The same for the kernel whose operands arrive packed (packed_kernels.hip): levels [level0, level1) of trees, bit for bit the
// results of the gathering kernel, or steps of a recurrence; always with an offset table.  Instances for recurrences cut the
// contraction into different numbers of slices, so the last bits of a sequence depend on the one that its batch takes.
constexpr double kPackedMaxBytes = 4294967296.0 - 131072.0;
// `variant`: instances with more or fewer units a workgroup (0 for trees); packed_variant picks one for a recurrence's batch.
int packed_groups(CellEpilogue epi, int32_t H, int32_t K, int32_t variant, int32_t n_cu);
int packed_members(CellEpilogue epi, int32_t H, int32_t variant);  // workgroups of a group (n_cb)
int packed_variant(CellEpilogue epi, int32_t H, int32_t n_live, int32_t directions, int32_t n_cu);
hipError_t launch_packed(CellEpilogue epi, const StationaryArgs& s, hipStream_t stream, const LaunchEvents& ev = LaunchEvents());

// States of tree nodes that other kernels have stored go to their places: list positions [0, n).
struct PackStatesArgs {
  int32_t n, H;
  const int32_t* rows; const int32_t* place;
  const float* h; const float* c;
  void* operand; float* cells;
};
hipError_t launch_pack_states(const PackStatesArgs& p, hipStream_t stream, const LaunchEvents& ev = LaunchEvents());

}  // namespace acrobat
