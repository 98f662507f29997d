// Deals random forests out to groups and checks the lists that the weight-stationary kernel walks: every internal node
// appears once, in its own level and in its tree's group; the offset table is complete; a group's levels only get
// narrower, and a node's children that are internal belong to earlier levels of the same group.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <string>
#include <vector>

#include "scheduler.h"

using namespace acrobat;

namespace {
uint64_t state = 88172645463325252ull;
int rnd_in(int lo, int hi) {
  state ^= state << 13; state ^= state >> 7; state ^= state << 17;
  return lo + (int)((state >> 32) % (uint64_t)(hi - lo + 1));
}
#define CHECK(cond) \
  do { if (!(cond)) { std::printf("CHECK failed: %s (line %d)\n", #cond, __LINE__); std::exit(1); } } while (0)

// random shape: two random subtrees are joined until one is left (leaves first, children before parents)
void add_tree(std::vector<int32_t>& off, std::vector<int32_t>& l, std::vector<int32_t>& r, int leaves) {
  std::vector<int> open;
  for (int i = 0; i < leaves; ++i) { open.push_back(i); l.push_back(-1); r.push_back(-1); }
  for (int id = leaves; open.size() > 1; ++id) {
    int pick[2];
    for (int& p : pick) {
      const int at = rnd_in(0, (int)open.size() - 1);
      p = open[at];
      open.erase(open.begin() + at);
    }
    l.push_back(pick[0]);
    r.push_back(pick[1]);
    open.push_back(id);
  }
  off.push_back((int32_t)l.size());
}
}  // namespace

int main() {
  TreeScheduler scheduler;
  TreeGrouping grouping;
  TreeSchedule s;
  for (int round = 0; round < 300; ++round) {
    std::vector<int32_t> off{0}, l, r;
    const int n_trees = rnd_in(1, 40), most = rnd_in(1, 60);
    for (int t = 0; t < n_trees; ++t) add_tree(off, l, r, rnd_in(1, most));
    const int N = off.back();
    std::vector<int32_t> token((size_t)N, 0);
    const acrobat_trees trees{n_trees, off.data(), l.data(), r.data(), token.data()};
    std::string err;
    CHECK(scheduler.begin(trees, 1, s, nullptr, err) == ACROBAT_OK);
    scheduler.finish(trees, s);
    const int n_leaf = s.level_off[1], L = s.n_levels;
    if (n_leaf == N) continue;
    const int groups = rnd_in(1, rnd_in(0, 1) ? 256 : 8);
    const int32_t kUnset = -77;
    std::vector<int32_t> out(N, kUnset), a(N, kUnset), b(N, kUnset), table((size_t)L * groups + 1, kUnset);
    const bool in_order = rnd_in(0, 1) != 0;
    grouping.stage(trees, s, groups, in_order, out.data(), a.data(), b.data(), table.data());
    for (int p = 0; p < n_leaf; ++p) CHECK(out[p] == kUnset);  // the leaf lists are someone else's
    std::vector<int> group_of_tree(n_trees, -1), level_of(N, 0), seen(N, 0), tree_of(N);
    for (int t = 0; t < n_trees; ++t)
      for (int g = off[t]; g < off[t + 1]; ++g) tree_of[g] = t;
    for (int lv = 1; lv < L; ++lv)
      for (int p = s.level_off[lv]; p < s.level_off[lv + 1]; ++p) level_of[s.level_nodes[p]] = lv;
    CHECK(table[(size_t)L * groups] == N);
    std::vector<int> width(groups, 1 << 30), size(groups, 0);
    for (int lv = 1; lv < L; ++lv)
      for (int g = 0; g < groups; ++g) {
        const int p0 = table[(size_t)lv * groups + g], p1 = table[(size_t)lv * groups + g + 1];
        CHECK(p0 >= s.level_off[lv] && p0 <= p1 && p1 <= s.level_off[lv + 1]);
        CHECK(p1 - p0 <= width[g]);
        width[g] = p1 - p0;
        for (int p = p0; p < p1; ++p) {
          const int id = out[p], t = tree_of[id], base = off[t];
          CHECK(level_of[id] == lv && !seen[id] && (p == p0 || out[p - 1] < id));
          seen[id] = 1;
          ++size[g];
          CHECK(group_of_tree[t] < 0 || group_of_tree[t] == g);
          group_of_tree[t] = g;
          CHECK(a[p] == base + l[id] && b[p] == base + r[id]);
          CHECK(level_of[a[p]] < lv && level_of[b[p]] < lv);
        }
      }
    for (int g = 0; g < N; ++g) CHECK(seen[g] == (l[g] >= 0));
    for (int g = 0; g < groups; ++g)  // dealt out evenly
      CHECK(groups > n_trees || size[g] <= (in_order ? N / (2 * groups) : (N - n_leaf) / groups) + most);
    for (int t = 1, last = -1; in_order && t < n_trees; ++t) {
      if (group_of_tree[t - 1] >= 0) last = group_of_tree[t - 1];
      CHECK(group_of_tree[t] < 0 || group_of_tree[t] >= last);
    }
  }
  // sequences: every (step, sequence, direction) once, rows and previous rows in the direction of the steps, and position i
  // of a group's share the same sequence at every step
  for (int round = 0; round < 300; ++round) {
    const int n_seq = rnd_in(1, 60), directions = rnd_in(1, 2);
    std::vector<int32_t> len(n_seq), row0(n_seq);
    int R = 0, T = 0;
    for (int q = 0; q < n_seq; ++q) {
      len[q] = rnd_in(0, 12);
      row0[q] = R;
      R += len[q];
      T = len[q] > T ? len[q] : T;
    }
    if (T == 0) continue;
    const int groups = directions * rnd_in(1, 20);
    std::vector<int32_t> out((size_t)directions * R, -1), off((size_t)T * groups + 1, -1);
    stage_seq_groups(n_seq, len.data(), T, groups, directions, out.data(), off.data());
    CHECK(off[0] == 0 && off[(size_t)T * groups] == directions * R);
    std::vector<int> seen((size_t)directions * R, 0);
    std::vector<int> seq_of(R);
    for (int q = 0; q < n_seq; ++q)
      for (int t = 0; t < len[q]; ++t) seq_of[row0[q] + t] = q;
    for (int g = 0; g < groups; ++g) {
      std::vector<int> at;
      for (int t = 0; t < T; ++t) {
        const int p0 = off[(size_t)t * groups + g], p1 = off[(size_t)t * groups + g + 1];
        CHECK(p0 <= p1 && (t == 0 || p1 - p0 <= (int)at.size()));
        std::vector<int> now;
        for (int p = p0; p < p1; ++p) {
          const bool backward = directions == 2 && (g & 1);
          const int row = out[p], q = seq_of[row];
          CHECK(row == (backward ? row0[q] + len[q] - 1 - t : row0[q] + t));
          CHECK(t == 0 || at[p - p0] == q);
          CHECK(!seen[(size_t)backward * R + row]++);
          now.push_back(q);
        }
        at = now;
      }
    }
    for (int v : seen) CHECK(v == 1);
  }
  std::printf("grouping: ok\n");
  return 0;
}
