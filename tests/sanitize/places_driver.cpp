// Places of packed operands: in random forests dealt out to groups, and in random batches of sequences, every node's place
// is the row and side at which its one reader looks for it, no two nodes share one, blocks of two shares never meet, and the
// leaves are all listed once, with their tokens.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "scheduler.h"

using namespace acrobat;

namespace {
uint64_t state = 1181783497276652981ull;
int rnd_in(int lo, int hi) {
  state ^= state << 13; state ^= state >> 7; state ^= state << 17;
  return lo + (int)((state >> 32) % (uint64_t)(hi - lo + 1));
}
#define CHECK(cond) \
  do { if (!(cond)) { std::printf("CHECK failed: %s (line %d)\n", #cond, __LINE__); std::exit(1); } } while (0)

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

void trees_round(TreeScheduler& scheduler, TreeGrouping& grouping) {
  std::vector<int32_t> off{0}, l, r;
  const int n_trees = rnd_in(1, 40), most = rnd_in(1, 80);
  for (int t = 0; t < n_trees; ++t) add_tree(off, l, r, rnd_in(1, most));
  const int N = off.back();
  std::vector<int32_t> token((size_t)N);
  for (int i = 0; i < N; ++i) token[i] = rnd_in(0, 99);
  const acrobat_trees trees{n_trees, off.data(), l.data(), r.data(), token.data()};
  std::string err;
  TreeSchedule s;
  std::vector<int32_t> leaf_tokens;
  CHECK(scheduler.begin(trees, 100, s, &leaf_tokens, err) == ACROBAT_OK);
  scheduler.finish(trees, s);
  const int n_leaf = s.level_off[1], L = s.n_levels;
  if (n_leaf == N) return;
  const int groups = rnd_in(1, 12), first = rnd_in(0, 2) ? 1 : rnd_in(1, L - 1);
  std::vector<int32_t> out(N, -7), a(N, -7), b(N, -7), table((size_t)L * groups + 1), place(N, -7);
  grouping.stage(trees, s, groups, rnd_in(0, 1) != 0, out.data(), a.data(), b.data(), table.data());
  grouping.places(s, leaf_tokens, groups, first, out.data(), a.data(), b.data(), table.data(), place.data());
  const int p_first = s.level_off[first];
  std::set<int32_t> leaves, taken;
  for (int p = 0; p < n_leaf; ++p) {
    CHECK(out[p] >= 0 && out[p] < N && leaves.insert(out[p]).second);
    CHECK(a[p] == token[out[p]]);
  }
  std::map<int32_t, int32_t> place_of;
  for (int p = 0; p < N; ++p) {
    CHECK(place[p] >= -1);
    CHECK(place_of.emplace(out[p], place[p]).second);
    CHECK(place[p] < 0 || taken.insert(place[p]).second);
  }
  const int64_t blocks = share_blocks((int64_t)N - p_first, (int64_t)L * groups);
  std::set<int32_t> owned;
  int read = 0;
  for (int lv = first; lv < L; ++lv)
    for (int g = 0; g < groups; ++g) {
      const int share = lv * groups + g, p0 = table[share], p1 = table[share + 1];
      const int block = share_block(p0, p_first, share);
      for (int x = 0; x < (p1 - p0 + 15) / 16; ++x) CHECK(block + x < blocks && owned.insert(block + x).second);
      for (int p = p0; p < p1; ++p) {
        const int code = 2 * (16 * block + (p - p0));
        CHECK(place_of[a[p]] == code && place_of[b[p]] == code + 1);
        read += 2;
      }
    }
  CHECK((int)taken.size() == read);  // nobody else has a place
}

void sequences_round() {
  const int n_seq = rnd_in(1, 90), directions = rnd_in(1, 2);
  std::vector<int32_t> len((size_t)n_seq);
  int R = 0, T = 0;
  for (int32_t& v : len) { v = rnd_in(0, 12); R += v; T = T > v ? T : v; }
  if (T < 1) return;
  const int groups = directions * rnd_in(1, 6), E = directions * R;
  std::vector<int32_t> out(E), table((size_t)T * groups + 1);
  stage_seq_groups(n_seq, len.data(), T, groups, directions, out.data(), table.data());
  int second = 0;
  for (const int32_t v : len) second += v > 1;
  const int blocks = seq_share_blocks(second, groups / directions);
  for (int t = 0; t < T; ++t)
    for (int g = 0; g < groups; ++g) {
      const int share = t * groups + g, p0 = table[share], n = table[share + 1] - p0;
      CHECK(t == 0 || n <= 16 * blocks);  // (a first step reads no packed state)
      for (int i = 0; t > 0 && i < n; ++i) {  // row i of the step before left its state for row i, and its row is found from it
        const int prev = out[p0 + i] + (directions == 2 && (g & 1) ? 1 : -1);
        CHECK(i < table[share - groups + 1] - table[share - groups] && out[table[share - groups] + i] == prev);
      }
    }
}
}  // namespace

int main() {
  TreeScheduler scheduler;
  TreeGrouping grouping;
  for (int round = 0; round < 400; ++round) trees_round(scheduler, grouping);
  for (int round = 0; round < 400; ++round) sequences_round();
  std::printf("places: ok\n");
  return 0;
}
