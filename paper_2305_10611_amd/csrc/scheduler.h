// Host level scheduler: structures -> per-depth node lists (no GPU code here).
#pragma once
#include <cstdint>
#include <string>
#include <vector>

#include "acrobat.h"

namespace acrobat {

struct TreeSchedule {
  int32_t n_nodes = 0;
  int32_t n_trees = 0;
  int32_t n_levels = 0;
  std::vector<int32_t> level_off;    // [n_levels + 1]
  std::vector<int32_t> level_nodes;  // [N] global ids, ascending inside a level
  std::vector<int32_t> lrow, rrow;   // [N] global child ids by list position, -1 at leaves
};

// Returns ACROBAT_OK / EINVAL / ESTRUCT; `err` explains a failure.
int schedule_trees(const acrobat_trees& trees, int32_t vocab, TreeSchedule& out, std::string& err);

// The same schedule in two phases with buffers that live across calls (a context owns one of these), so that
// a forward call can launch level 0 while the host is still sorting the internal levels:
//  begin()  validates the whole structure (nothing may be launched for malformed input), computes every
//           node's depth, level_off, and the level-0 list: out.level_nodes[0 .. n_leaf) = the leaves by
//           ascending id, their tokens in leaf_tokens (if not null; needs trees.token);
//  finish() fills level_nodes / lrow / rrow of the internal levels.
// `out` is resized, never shrunk to fit: its vectors keep their capacity from call to call.
class TreeScheduler {
 public:
  int begin(const acrobat_trees& trees, int32_t vocab, TreeSchedule& out, std::vector<int32_t>* leaf_tokens, std::string& err);
  void finish(const acrobat_trees& trees, TreeSchedule& out);

 private:
  int general_tree(const acrobat_trees& tr, int32_t t, int32_t vocab, std::string& err);
  std::vector<int32_t> depth_, parent_, cursor_, count_;
  std::vector<uint8_t> mark_;  // fast path: "has a parent"; general path: children still to come
};

// Deals whole trees out to groups that run their internal levels independently of each other, and lists every internal
// level group by group.  Trees by descending size go to the groups in turn, back and forth (0 .. g-1, g-1 .. 0, ...), so
// the groups get alike numbers of nodes and alike tallest trees; or (in_order) a group gets consecutive trees, as nearly an
// even share of the nodes as whole trees allow, which leaves the lists as the schedule has them and costs the host little.
class TreeGrouping {
 public:
  // Writes the lists of the internal levels, positions [level_off[1], N): row written, left and right child rows; inside
  // a level by group, inside a group by ascending id.  off[lv * groups + g] is the first position of group g's share of
  // level lv >= 1 (entries of level 0: its end), off[n_levels * groups] = N.
  void stage(const acrobat_trees& trees, const TreeSchedule& s, int32_t groups, bool in_order, int32_t* out, int32_t* left,
             int32_t* right, int32_t* off);
  // Places for groups that run levels first .. n_levels - 1 of the staged lists: share (lv, g) of those has blocks of 16 rows
  // from share_block() on, and the node in row r of block b reads places 2 (16 b + r) (left) and one more (right).  place[p]
  // of every list position: where its parent reads it, -1 if nobody does.  The leaves are listed here as well, positions
  // [0, level_off[1]): out = row written, left = token, in the order of their places - a block's left children, then its right
  // ones, so that neighbours in the list go to neighbouring rows of an operand - and behind them those without a place.
  void places(const TreeSchedule& s, const std::vector<int32_t>& leaf_tokens, int32_t groups, int32_t first, int32_t* out,
              int32_t* left, const int32_t* right, const int32_t* off, int32_t* place);

 private:
  std::vector<int32_t> position_;  // of every node: of a leaf in level_nodes, of others in the lists
  std::vector<int32_t> order_, count_;
  std::vector<uint8_t> group_;  // of every node (at most 256 groups)
};

struct SeqSchedule {
  int64_t n_rows = 0;
  int32_t n_levels = 0;
  std::vector<int32_t> level_off;   // [n_levels + 1]
  std::vector<int32_t> level_rows;  // [sum len]
};

int schedule_seqs(int32_t n_seq, const int32_t* len, SeqSchedule& out, std::string& err);

// First block of 16 rows of a share that starts at list position p0: counted from position `base`, share number
// level * groups + group.  Rounding down, with a block to spare for every share, keeps them apart.
inline int32_t share_block(int32_t p0, int32_t base, int32_t share) { return (p0 - base) / 16 + share; }
// Blocks that shares numbered below n_shares of n list positions may take up.
inline int64_t share_blocks(int64_t n, int64_t n_shares) { return n / 16 + n_shares + 1; }
// Blocks of 16 rows that hold any share of a step behind the first, n_second nodes in the second step of a direction that is
// dealt out to `lists` lists.
inline int32_t seq_share_blocks(int32_t n_second, int32_t lists) { return ((n_second + lists - 1) / lists + 15) / 16; }

// Deals sequences out to groups that run their recurrences independently of each other (by descending length, back and
// forth) and lists every step group by group.  Step t of sequence s writes row seq_off[s] + t and reads the row before it
// (directions == 2: odd groups list the backward direction, which starts at the last row and reads the row behind).
// out: directions * (sum len) entries.
// off[t * groups + g]: first position of group g's share of step t, off[n_steps * groups] the end.
// A group's share of a step lists the first sequences of its share of the step before, in the same order.
void stage_seq_groups(int32_t n_seq, const int32_t* len, int32_t n_steps, int32_t groups, int32_t directions, int32_t* out,
                      int32_t* off);

// Bidirectional RNN with an output phase: levels 0 .. max len - 1 hold step k of both directions
// (codes: forward row, then R + backward row), the last level holds every output operator (2R + row).
struct BirnnSchedule {
  int64_t n_rows = 0;
  int32_t n_levels = 0;              // max len + 1, or 0
  std::vector<int32_t> level_off;    // [n_levels + 1] into level_codes
  std::vector<int32_t> level_codes;  // [3 R]
  std::vector<int32_t> fwd_off;      // [max len + 1]: forward entries of level k are
                                     // level_codes[level_off[k] .. level_off[k] + fwd_off[k+1] - fwd_off[k])
};

int schedule_birnn(int32_t n_seq, const int32_t* len, BirnnSchedule& out, std::string& err);

}  // namespace acrobat
