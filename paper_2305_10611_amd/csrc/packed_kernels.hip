// Weight-stationary cell kernels whose operands arrive packed (gfx950): whole recurrences and the grouped internal
// levels of tree batches in one launch.
//
// As in tree_kernels.hip a group of workgroups keeps the weights of a cell in its registers and node rows stream past
// them.  There the rows are gathered from the state arena, which is what bounded a level: a matrix instruction wants
// neighbouring lanes to hold DIFFERENT rows, and a load whose neighbouring lanes are in different rows fetches 37 KB/us per
// compute unit where one that reads 1 KB in a row fetches 126 (64 KB out of the XCD's L2; turning rows through LDS instead
// made the chain of a level longer than the loads it saved: 2.9 -> 3.7 us at H = 256).  Every state has exactly one reader
// in these batches - a tree node its parent, a step of a sequence the next - so here the workgroup that makes a state
// stores it a second time, split into its two fp16 terms, at its PLACE: its row in the matrix operand of the block of 16
// nodes that its reader belongs to, in the order in which the lanes want it.  The reader's loads are then contiguous, and
// nothing is left to convert.  c states travel the same way (`cells`), so that a level starts without any index list.
// Bound: narrow levels and steps by their chain - announcement 0.9, operand 0.6, matrix instructions and sums 0.5, gates and
// stores 0.5 us -, wide levels by the matrix cores (7 186 rows, H = 512: 102 us, 1.1 PFLOP/s of fp16 products; a large
// library product reaches 1.3).  Forward calls against the gathering kernel: 8 trees of 20 leaves, H = 256 50 -> 43 us, 64
// trees 91 -> 84; LSTM, 256 sequences, H = 512 528 -> 382 (with packed input rows), 75 sequences, H = 320 229 -> 157; BiRNN, 600 sequences, H = 256
// 214 -> 175.  A recurrence needs no list of places or previous rows: a share's sequences are the first ones of the share
// before, so the words that a call uploads are as many as its rows.
//
// Operand: blocks of 16 rows; a 32-k step of a block is 64 lanes x 16 bytes of hi terms, then the same of lo terms; lane
// l holds row l % 16, k = 4 (l / 16) + 0 .. 3 and 16 more.  A tree node has its left child's H columns, then its right
// child's.  cells: [block][side][workgroup of the group][row][unit].  Share (level, group) of a tree batch, list positions p0
// ..., has the blocks from (p0 - first_position) / 16 + level * groups + group on (rounded down: no two shares meet).  A
// recurrence has `sets` sets of blocks, at least two, and in each a group those of its widest share: step t reads set t % sets
// and leaves its states in the next one, which only steps before it have read - all of a group has announced those before it
// starts on t.  (A set for every step was slower where they outgrew the caches, LSTM, 256 sequences of 1 to 100 steps, H = 512
// 439 against 386 us, and a little faster where they are small, 75 of 1 to 60, H = 320 160 against 163; keeping c states of single
// blocks in registers changed nothing.)
// Tree levels: the arithmetic of the gathering kernel, in the same order, so the same bits.
#include "tree_kernels.h"

#include "cell_epilogue.h"
#include "packed_rows.h"
#include "split_fp16.h"

#include <algorithm>
#include <atomic>
#include <type_traits>

namespace acrobat {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

// What a workgroup holds and does between two barriers.  NW wavefronts are CH blocks of 16 hidden units x KS slices of the
// contraction; a wavefront has G column tiles of 16: the gates of its units or, for a cell with one gate, G blocks of units.
// RB blocks of 16 rows are multiplied between two barriers, after which each thread finishes EPT elements (all G tiles of
// each).  Partial sums of a wavefront and row block: [row][unit] vectors of the first four tiles, then the fifth.
template <int G, int NW, int NS, int RB, int CH>
struct PackedShape {
  static constexpr int KS = NW / CH;
  static constexpr int ZV = G == 1 ? 0 : 1024, ZQ = ZV + (G == 5 || G == 1 ? 256 : 0);
  static constexpr int EPT = RB * CH * 4 / NW;
  static constexpr int RR = RB * NS <= 4 ? RB : 1;                               // blocks whose operands are in flight
  static constexpr int ZB = 2 * RB * NW * ZQ * (int)sizeof(float) <= 82 * 1024 ? 2 : 1;  // buffers of partial sums
  static constexpr size_t kLdsBytes = (size_t)ZB * RB * NW * ZQ * sizeof(float);
  static_assert(EPT >= 1 && RB * CH * 4 % NW == 0, "every thread finishes elements");
  static_assert(ZB * RB * ZQ >= kTurnFloats, "weights are turned where the partial sums go afterwards");
  static_assert(CH == 1 || (CH == NW / 4 && RB == 1), "256 threads finish a row block of a unit block");
};

template <int G, int EPI, int NW, int NS, int RB, int CH>
__global__ __launch_bounds__(64 * NW, 2) void cell_packed_kernel(const StationaryArgs s) {
  using S = PackedShape<G, NW, NS, RB, CH>;
  constexpr bool kTree = EPI == EPI_TREE_INTERNAL, kTiles = EPI == EPI_RNN_STEP;  // kTiles: the G tiles are blocks of units
  constexpr int KS = S::KS, ZV = S::ZV, ZQ = S::ZQ, EPT = S::EPT, RR = S::RR;
  extern __shared__ __attribute__((aligned(16))) float zbuf[];  // [ZB][RB][NW][ZQ]
  __shared__ float s_bias[CH][G][16];
  __shared__ __attribute__((aligned(16))) float s_winv[NW][16][4];
  __shared__ float s_winv4[NW][16];
  __shared__ int s_go;

  // workgroup ids that agree modulo 8 share an XCD (placement only matters for speed)
  const int slot = blockIdx.x >> 3;
  const int group = (slot / s.n_cb) * 8 + (blockIdx.x & 7), cb = slot % s.n_cb;
  if (group >= s.n_groups) return;
  const CellLevelArgs& a = s.a[s.two ? group & 1 : 0];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ks = w % KS, ch = w / KS;
  const int li = lane & 15, kq = lane >> 4;
  const int H = a.H, K = a.nseg * a.kseg, T = K >> 5;  // 32-k steps, at most KS * NS
  // first weight row of tile g of unit block c of this workgroup; a cell with one gate has no other rows
  const auto tile_row = [&](int g, int c) { return kTiles ? 16 * (cb * G + g) : gate_row<EPI>(g) * H + 16 * (cb * CH + c); };

  // The lists are cold memory, and a level's would come a microsecond late each time: while the weights are under way the
  // workgroups of the group bring the first 128 rows of every level's share into their L2.
  int touched = 0;
  if (s.level1 - s.level0 > 1) {
    const int* const list = kTree && (cb & 1) ? s.place : a.out_rows;
    for (int l = s.level0 + (tid >> 2); l < s.level1; l += 16 * NW) {
      const int p = s.off[l * s.n_groups + group] + 32 * (tid & 3);
      if (p < s.off[l * s.n_groups + group + 1]) touched |= list[p];
    }
  }

  // ---- this wavefront's weights: tile g, column li, steps ks + KS t, fetched line by line and turned through LDS
  half8 whi[G][NS], wlo[G][NS];
  {
    floatx4 raw[G][NS][2];  // (every load in flight at once)
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const float* row = a.W + (size_t)(tile_row(g, ch) + (lane >> 3)) * (size_t)a.ldw + 4 * (lane & 7);
#pragma unroll
      for (int t = 0; t < NS; ++t) {
        const int step = ks + KS * t;
        raw[g][t][0] = raw[g][t][1] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        if (step < T) {
          raw[g][t][0] = *reinterpret_cast<const floatx4*>(row + 32 * step);
          raw[g][t][1] = *reinterpret_cast<const floatx4*>(row + 8 * (size_t)a.ldw + 32 * step);
        }
      }
    }
    float* const tile = zbuf + w * kTurnFloats;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      float sc[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        float m = 0.0f;
#pragma unroll
        for (int t = 0; t < NS; ++t) m = largest(raw[g][t][h], m);
        sc[h] = scale_for(largest_of_line(m));
        if ((lane & 7) == 0) {
          float unit = inverse_power(sc[h]) * (1.0f / kStateScale);
          if (unit > kLargestUnit) unit = __builtin_inff();  // (the sums are not finite then)
          const int col = (lane >> 3) + 8 * h;
          if (g < 4 && G > 1) s_winv[w][col][g] = unit;
          else s_winv4[w][col] = unit;
        }
      }
      if (ks == 0 && lane < 16) s_bias[ch][g][li] = a.bias ? a.bias[tile_row(g, ch) + li] : 0.0f;
#pragma unroll
      for (int t = 0; t < NS; ++t) {
        turn_write(tile, lane, raw[g][t], sc[0], sc[1]);
        turn_read(tile, lane, whi[g][t], wlo[g][t]);
      }
    }
  }
  asm volatile("" ::"v"(touched));

  // ---- the elements this thread finishes: row er of row blocks rb0, rb0 + NW / 4, ... of a chunk, unit j (of tile g, if
  // tiles are units: j + 16 g)
  const int rb0 = CH > 1 ? 0 : w >> 2, my_ch = CH > 1 ? w >> 2 : 0;
  const int jb = kTiles ? cb * G : cb * CH + my_ch;  // its (first) block of 16 units
  const int er = (tid & 255) >> 4, eu = tid & 15, j = 16 * jb + eu;
  const __amdgpu_buffer_rsrc_t operand = agent_buffer(s.operand, s.operand_bytes);
  const unsigned block_bytes = 64u * K;  // of the operand
  constexpr unsigned kNowhere = 0xfffff000u;  // past the end of the buffer: reads zeros, stores nothing
  constexpr unsigned kNoBlock = kNowhere - 2048u * KS * NS;
  const auto z_at = [&](int g) { return g < 4 && G > 1 ? (er * 16 + eu) * 4 + g : ZV + er * 16 + eu; };  // partial sums of tile g
  // where a state of unit 16 b + eu goes inside its row's place
  const auto in_place = [&](int b) { return 2048u * (b >> 1) + 8u * (b & 1) + 512u * (eu & 2) + 256u * (eu >> 2) + 4u * (eu & 1); };
  const unsigned cell_at = 1024u * jb + 4u * (tid & 255);  // of such an element inside (block, side) of cells
  ACROBAT_GLOBAL int* const out_rows = keep(const_cast<int*>(a.out_rows));
  ACROBAT_GLOBAL int* const place = keep(const_cast<int*>(s.place));
  // (read with scalar loads: nothing in the launch writes it)
  const __attribute__((address_space(4))) int* const offsets = (const __attribute__((address_space(4))) int*)s.off;
  ACROBAT_GLOBAL float* const zadd = keep(const_cast<float*>(a.zadd));
  ACROBAT_GLOBAL float* const h_rows = keep(a.h);
  ACROBAT_GLOBAL float* const c_rows = keep(a.c);
  ACROBAT_GLOBAL float* const cells = keep(s.cells);
  unsigned* const counter = s.counters + (size_t)group * kTreeCounterStride;

  floatx4 ring[RR][NS][2];  // operand steps under way: hi, lo
  auto request = [&](unsigned at, int r, int t) {
    const int step = ks + KS * t;
    at = step < T ? at + 2048u * step : kNowhere;
    ring[r][t][0] = load_agent_f4(operand, at + 16u * lane);
    ring[r][t][1] = load_agent_f4(operand, at + 16u * lane + 1024u);
  };
  auto share_of = [&](int lv, int& p0, int& p1) {
    p0 = offsets[lv * s.n_groups + group];
    p1 = offsets[lv * s.n_groups + group + 1];
  };
  // rows written, and of tree nodes the places, of this thread's rows; for a recurrence, whose addends they name, a chunk ahead
  int out[EPT], to[EPT], next_out[EPT];
  auto request_lists = [&](int (&o)[EPT], int p, int end) {  // tail rows repeat the last node; never stored
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      int i = p + 16 * (rb0 + e * (NW / 4)) + er;
      i = i < end ? i : end - 1;
      o[e] = at_byte(out_rows, 4u * (unsigned)i);
      if constexpr (kTree) to[e] = at_byte(place, 4u * (unsigned)i);
    }
  };

  int lv = s.level0, p0, p1;
  unsigned arrived = 0;  // levels this group has announced
  // recurrences: first block of the set that this step reads, and of the one after it
  const unsigned set_blocks = (unsigned)s.n_groups * (unsigned)s.share_blocks, set0 = (unsigned)group * (unsigned)s.share_blocks;
  const unsigned sets_end = set0 + (unsigned)s.sets * set_blocks;
  unsigned here = kTree ? 0u : set0 + (unsigned)(lv % s.sets) * set_blocks, there = here + set_blocks;
  if (there == sets_end) there = set0;
  share_of(lv, p0, p1);
  if (p0 >= p1) return;  // (nothing in this level: nothing in a later one)
  if constexpr (!kTree) request_lists(next_out, p0, p1);
  __syncthreads();

  // One level; false when there is nothing more to do.  kFirst: step 0 of a recurrence, whose states before it are zero or
  // (single gate) the row a.first.
  auto run_level = [&](auto first_level) -> bool {
    constexpr bool kFirst = decltype(first_level)::value;
    const int n = p1 - p0, nb = (n + 15) >> 4;
    int c0 = 0, c1 = 0;  // the next level's share
    if (lv + 1 < (kTree ? s.level1 : s.n_steps)) share_of(lv + 1, c0, c1);
    const unsigned block0 = kTree ? (unsigned)((p0 - s.first_position) >> 4) + (unsigned)(lv * s.n_groups + group) : here;
    // a share's sequences are a prefix of the step before's: row i of a block is read as row i of the same block of the other set
    const unsigned reader0 = there;
    float p[EPT][2], zx[EPT][kTree ? 1 : G];
    auto take_lists = [&]() {
#pragma unroll
      for (int e = 0; e < EPT; ++e) out[e] = next_out[e];
    };
    auto fetch_addends = [&]() {  // cold memory: requested before the wait
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        if constexpr (EPI == EPI_LSTM_STEP) {
#pragma unroll
          for (int g = 0; g < G; ++g) zx[e][g] = zadd[(size_t)out[e] * (size_t)(G * H) + g * H + j];
        }
        if constexpr (kTiles) {
#pragma unroll
          for (int g = 0; g < G; ++g) zx[e][g] = zadd[(size_t)out[e] * (size_t)H + 16 * g + j];
        }
      }
    };
    auto fetch_cells = [&](int b, bool all) {  // (stored by this workgroup, or by an earlier launch)
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        // (a chunk of one row block: the others' elements are fetched from it as well, and not used)
        const unsigned block = block0 + b + (all ? rb0 + e * (NW / 4) : 0);
        p[e][0] = p[e][1] = 0.0f;
        if constexpr (kTree || (EPI == EPI_LSTM_STEP && !kFirst)) p[e][0] = at_byte(cells, block * block_bytes + cell_at);
        if constexpr (kTree) p[e][1] = at_byte(cells, block * block_bytes + 64u * H + cell_at);
      }
    };
    if constexpr (!kTree) {
      take_lists();
      fetch_addends();
    }
    if (arrived > 0) {  // the group's previous level is complete once all its workgroups have announced it
      if (tid == 0) s_go = wait_for(counter, (unsigned)s.n_cb * arrived, s.status, s.max_polls) ? 1 : 0;
      __syncthreads();
      if (!s_go) return false;
    }
    auto block_at = [&](int b) { return b < nb ? (block0 + b) * block_bytes : kNoBlock; };
    if constexpr (!kFirst) {
#pragma unroll
      for (int r = 0; r < RR; ++r)
#pragma unroll
        for (int t = 0; t < NS; ++t) {
          request(block_at(r), r, t);
          hold_order();
        }
    }
    fetch_cells(0, nb >= RB);

    // Row blocks b .. b + blocks - 1 of the level
    auto chunk = [&](const int b, auto n_blocks) {
      constexpr int blocks = decltype(n_blocks)::value;
      const bool more = b + blocks < nb;
      if constexpr (kTree) request_lists(out, p0 + 16 * b, p1);  // (behind the loads of this chunk: they return in order)
      float* const zc = zbuf + (S::ZB == 2 ? (b / RB & 1) * (RB * NW * ZQ) : 0);
#pragma unroll
      for (int r = 0; r < blocks; ++r) {
        floatx4 acc[G];
#pragma unroll
        for (int g = 0; g < G; ++g) acc[g] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        auto multiply = [&](const half8 hi, const half8 lo, int t) {
#pragma unroll
          for (int g = 0; g < G; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(lo, whi[g][t], acc[g], 0, 0, 0);
#pragma unroll
          for (int g = 0; g < G; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hi, wlo[g][t], acc[g], 0, 0, 0);
#pragma unroll
          for (int g = 0; g < G; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hi, whi[g][t], acc[g], 0, 0, 0);
        };
        if constexpr (!kFirst) {
          const unsigned next = block_at(b + r + RR);
          constexpr int slot = 0;
#pragma unroll
          for (int t = 0; t < NS; ++t) {
            floatx4(&x)[2] = ring[RR == RB ? r : slot][t];
            multiply(__builtin_bit_cast(half8, x[0]), __builtin_bit_cast(half8, x[1]), t);
            hold_order();
            request(next, RR == RB ? r : slot, t);
            hold_order();
          }
        } else if constexpr (kTiles) {
#pragma unroll
          for (int t = 0; t < NS; ++t) {
            const int step = ks + KS * t;
            if (step < T) {
              half8 hi, lo;
              split8(*reinterpret_cast<const floatx4*>(a.first + 32 * step + 4 * kq),
                     *reinterpret_cast<const floatx4*>(a.first + 32 * step + 16 + 4 * kq), kStateScale, hi, lo);
              multiply(hi, lo, t);
            }
          }
        }
        float* const z = zc + (r * NW + w) * ZQ;
        if constexpr (G > 1) {
          const floatx4 unit = *reinterpret_cast<const floatx4*>(s_winv[w][li]);
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            floatx4 part = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int g = 0; g < (G < 4 ? G : 4); ++g) part[g] = acc[g][v] * unit[g];
            *reinterpret_cast<floatx4*>(z + ((4 * kq + v) * 16 + li) * 4) = part;
          }
        }
        if constexpr (G == 5 || G == 1) {
          const float unit = s_winv4[w][li];
#pragma unroll
          for (int v = 0; v < 4; ++v) z[ZV + (4 * kq + v) * 16 + li] = acc[G - 1][v] * unit;
        }
      }
      // what comes next: behind this chunk's own loads, which would otherwise wait (loads return in order)
      if constexpr (!kTree)
        request_lists(next_out, more ? p0 + 16 * (b + blocks) : c0 < c1 ? c0 : p0, more ? p1 : c0 < c1 ? c1 : p1);
      // (one of two buffers has been read two chunks later: its readers have passed the barrier in between)
      __syncthreads();
      float zs[EPT][G];
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const int r = rb0 + e * (NW / 4);
        if (r >= blocks) continue;  // (a chunk of one row block: half of the threads have nothing to finish)
        float* const zr = zc + (r * NW + my_ch * KS) * ZQ;
        if constexpr (G > 1) {
          floatx4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int q = 0; q < KS; ++q) {
            const floatx4 part = *reinterpret_cast<const floatx4*>(zr + q * ZQ + (er * 16 + eu) * 4);
#pragma unroll
            for (int g = 0; g < 4; ++g) sum[g] += part[g];
          }
#pragma unroll
          for (int g = 0; g < (G < 4 ? G : 4); ++g) zs[e][g] = sum[g];
        }
        if constexpr (G == 5 || G == 1) {
          float sum = 0.0f;
#pragma unroll
          for (int q = 0; q < KS; ++q) sum += zr[q * ZQ + ZV + er * 16 + eu];
          zs[e][G - 1] = sum;
        }
        const bool live = 16 * (b + r) + er < n;
        float finite = 0.0f;
#pragma unroll
        for (int g = 0; g < G; ++g) finite = __builtin_fmaf(zs[e][g], 0.0f, finite);
        if (__builtin_expect(live && finite != 0.0f, 0)) {
          // What is not finite, or not to be split, is computed in fp32 from the arena's rows.  (Through LDS, this thread's
          // own words: indexed registers would cost spills in every block.)
          const __amdgpu_buffer_rsrc_t rsrc = agent_buffer(a.src0, s.src_bytes);
          unsigned at0 = 0u, at1 = 0u;
          if constexpr (kTree) {
            const int pos = p0 + 16 * (b + r) + er;
            at0 = (unsigned)a.idx0[pos] * (unsigned)a.ld0 * 4u;
            at1 = (unsigned)a.idx1[pos] * (unsigned)a.ld0 * 4u - 4u * a.kseg;
          } else if constexpr (!kFirst) {
            at0 = at1 = (unsigned)(s.two && (group & 1) ? out[e] + 1 : out[e] - 1) * (unsigned)a.ld0 * 4u;
          }
          const int k_end = kFirst && EPI == EPI_LSTM_STEP ? 0 : K;  // (no state before the first step: no product)
#pragma unroll
          for (int g = 0; g < G; ++g) zr[z_at(g)] = zs[e][g];
#pragma unroll 1
          for (int g = 0; g < G; ++g) {
            float* const at = zr + z_at(g);
            if (__builtin_isfinite(*at)) continue;
            const float* const wr = a.W + (size_t)(tile_row(g, my_ch) + eu) * (size_t)a.ldw;
            float sum = 0.0f;
#pragma unroll 1
            for (int k = 0; k < k_end; k += 4) {
              floatx4 x;
              if constexpr (kFirst) x = *reinterpret_cast<const floatx4*>(a.first + k);
              else x = load_agent_f4(rsrc, (k < a.kseg ? at0 : at1) + 4u * k);
              const floatx4 wk = *reinterpret_cast<const floatx4*>(wr + k);
#pragma unroll
              for (int c = 0; c < 4; ++c) sum = __builtin_fmaf(x[c], wk[c], sum);
            }
            *at = sum;
          }
#pragma unroll
          for (int g = 0; g < G; ++g) zs[e][g] = zr[z_at(g)];
        }
      }
      if (S::ZB == 1 && more) __syncthreads();  // the partial sums have been read
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const int r = rb0 + e * (NW / 4);
        if (r >= blocks || 16 * (b + r) + er >= n) continue;
        // a tree node's place: twice row + 16 block, and the side
        const bool read = kTree ? to[e] >= 0 : 16 * (b + r) + er < c1 - c0;
        const unsigned row = kTree ? (unsigned)to[e] >> 1 & 15u : (unsigned)er;
        const unsigned side_block = kTree ? 2u * (unsigned)(to[e] >> 5) + ((unsigned)to[e] & 1u) : reader0 + b + r;
        const unsigned place_at = side_block * (64u * H) + 16u * row;
        const unsigned row_at = 4u * ((unsigned)out[e] * (unsigned)H + j);
        const auto store_state = [&](float h, int b16, unsigned at) {
          const unsigned word = quad_word(split_state(h), lane);  // (a row's 16 lanes are live together)
          __builtin_amdgcn_raw_buffer_store_b32(word, operand, (int)(read ? place_at + in_place(b16) : kNowhere), 0, kAuxAgentScope);
          __hip_atomic_store(&at_byte(h_rows, at), h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };
        const auto bias = [&](int g) { return s_bias[my_ch][g][eu]; };
        if constexpr (kTiles) {
#pragma unroll
          for (int g = 0; g < G; ++g) store_state(fast_sigmoid(zs[e][g] + zx[e][g] + bias(g)), jb + g, row_at + 64u * g);
        } else {
          float c, h;
          if constexpr (kTree) {
            c = fast_sigmoid(zs[e][0] + bias(0)) * fast_tanh(zs[e][4] + bias(4)) + fast_sigmoid(zs[e][1] + bias(1)) * p[e][0] +
                fast_sigmoid(zs[e][2] + bias(2)) * p[e][1];
            h = fast_sigmoid(zs[e][3] + bias(3)) * fast_tanh(c);
          } else {
            c = fast_sigmoid(zs[e][1] + zx[e][1] + bias(1)) * p[e][0] +
                fast_sigmoid(zs[e][0] + zx[e][0] + bias(0)) * fast_tanh(zs[e][3] + zx[e][3] + bias(3));
            h = fast_sigmoid(zs[e][2] + zx[e][2] + bias(2)) * fast_tanh(c);
          }
          store_state(h, jb, row_at);
          at_byte(c_rows, row_at) = c;
          if (read) at_byte(cells, side_block * (64u * H) + 1024u * jb + 64u * row + 4u * eu) = c;
        }
      }
    };
    int b = 0;
    for (; b + RB <= nb; b += RB) {
      chunk(b, std::integral_constant<int, RB>());
      if (b + RB >= nb) break;
      if constexpr (!kTree) take_lists();
      fetch_cells(b + RB, b + 2 * RB <= nb);
      if constexpr (!kTree) fetch_addends();
    }
    if constexpr (RB > 1) {
      static_assert(RB == 2, "what is left is one block");
      if (nb & 1) chunk(nb - 1, std::integral_constant<int, 1>());
    }
    if (s.stamps && cb == 0 && tid == 0) s.stamps[lv * s.n_groups + group] = wall_clock64();
    const bool announce = lv + 1 < s.level1;
    if (announce) {
      wait_stores_done();  // this wavefront's stores have completed ...
      __syncthreads();     // ... and so have the other wavefronts'
      if (tid == 0) __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      ++arrived;
    }
    if (c0 >= c1 || !announce) return false;
    p0 = c0;
    p1 = c1;
    ++lv;
    if constexpr (!kTree) {
      here = there;
      there += set_blocks;
      if (there == sets_end) there = set0;
    }
    return true;
  };
  bool on = true;
  if constexpr (!kTree) {
    if (lv == 0) on = run_level(std::true_type());
  }
  while (on) on = run_level(std::false_type());
  if (arrived > 0 && tid == 0) leave_block(counter, s.n_cb);
}

// States that other kernels left in the arena go to their places: one wavefront per list position.
__global__ __launch_bounds__(256) void pack_states_kernel(const PackStatesArgs p) {
  const int lane = threadIdx.x & 63;
  const int i = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6);
  if (i >= p.n) return;
  const int to = p.place[i];
  if (to < 0) return;
  const size_t src = (size_t)p.rows[i] * p.H;
  const unsigned row = (unsigned)(to >> 1) & 15u, side_block = 2u * (unsigned)(to >> 5) + ((unsigned)to & 1u);
  unsigned char* const dst = static_cast<unsigned char*>(p.operand) + (size_t)side_block * (64u * p.H) + 16u * row;
  float* const cells = p.cells + (size_t)side_block * (16 * p.H) + 16 * row;
  for (int u = 4 * lane; u < p.H; u += 256) {  // four units, half of a 16-byte piece
    const floatx4 h = *reinterpret_cast<const floatx4*>(p.h + src + u);
    const floatx4 c = *reinterpret_cast<const floatx4*>(p.c + src + u);
    unsigned hi[2], lo[2];
    split4_packed(h, kStateScale, hi, lo);
    unsigned char* const at = dst + 2048u * (u >> 5) + 256u * ((u & 15) >> 2) + 8u * ((u >> 4) & 1);
    *reinterpret_cast<uintx2*>(at) = uintx2{hi[0], hi[1]};
    *reinterpret_cast<uintx2*>(at + 1024) = uintx2{lo[0], lo[1]};
    *reinterpret_cast<floatx4*>(cells + 256 * (size_t)(u >> 4) + (u & 15)) = c;
  }
}

template <int G, int EPI, int NW, int NS, int RB, int CH>
struct Packed {
  static constexpr size_t kLdsBytes = PackedShape<G, NW, NS, RB, CH>::kLdsBytes;
  static const void* kernel() { return reinterpret_cast<const void*>(&cell_packed_kernel<G, EPI, NW, NS, RB, CH>); }
  // More than 64 KB of dynamic LDS has to be asked for once per device (one bit per device id; two threads that both
  // find the bit clear both set the attribute, which is harmless).
  static hipError_t configure() {
    if (kLdsBytes <= 60 * 1024) return hipSuccess;
    static std::atomic<uint64_t> configured{0};
    int dev = 0;
    if (const hipError_t e = hipGetDevice(&dev); e != hipSuccess) return e;
    const uint64_t bit = 1ull << (dev & 63);
    if (dev < 64 && (configured.load(std::memory_order_acquire) & bit)) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute(kernel(), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBytes);
    if (e == hipSuccess && dev < 64) configured.fetch_or(bit, std::memory_order_release);
    return e;
  }
  static hipError_t launch(const StationaryArgs& s, hipStream_t stream, const LaunchEvents& ev) {
    if (const hipError_t e = configure(); e != hipSuccess) return e;
    const unsigned grid = 8u * (unsigned)s.n_cb * (unsigned)((s.n_groups + 7) / 8);
    launch_with_events((cell_packed_kernel<G, EPI, NW, NS, RB, CH>), dim3(grid), dim3(64 * NW), kLdsBytes, stream, ev.start, ev.stop, s);
    return hipGetLastError();
  }
  // workgroups of this kernel that a compute unit holds (0: the query failed); asked once per device, 1 to 2 us
  static int per_cu() {
    static std::atomic<int> known[64];  // one more than the answer
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) == hipSuccess && dev < 64)
      if (const int k = known[dev].load(std::memory_order_relaxed); k > 0) return k - 1;
    if (configure() != hipSuccess || hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel(), 64 * NW, kLdsBytes) != hipSuccess) {
      (void)hipGetLastError();
      return 0;
    }
    if (dev < 64) known[dev].store(n + 1, std::memory_order_relaxed);
    return n;
  }
};

// Calls f with the instance for K columns.  Tree levels: 16 units a workgroup, four wavefronts up to K = 512 and eight above, as
// the gathering kernel.  Recurrences: see packed_variant.
template <class F>
auto dispatch(CellEpilogue epi, int32_t H, int32_t K, int32_t variant, F&& f) {
  if (epi == EPI_TREE_INTERNAL) {
    if (K <= 128) return f(Packed<5, EPI_TREE_INTERNAL, 4, 1, 1, 1>());
    if (K <= 256) return f(Packed<5, EPI_TREE_INTERNAL, 4, 2, 1, 1>());
    if (K <= 512) return f(Packed<5, EPI_TREE_INTERNAL, 4, 4, 1, 1>());
    if (K <= 768) return f(Packed<5, EPI_TREE_INTERNAL, 8, 3, 2, 1>());
    return f(Packed<5, EPI_TREE_INTERNAL, 8, 4, 2, 1>());
  }
  if (epi == EPI_LSTM_STEP) {
    if (variant == 0) {
      if (K <= 128) return f(Packed<4, EPI_LSTM_STEP, 4, 1, 1, 1>());
      if (K <= 256) return f(Packed<4, EPI_LSTM_STEP, 4, 2, 1, 1>());
      if (K <= 384) return f(Packed<4, EPI_LSTM_STEP, 4, 3, 1, 1>());
      return f(Packed<4, EPI_LSTM_STEP, 4, 4, 1, 1>());
    }
    if (K <= 128) return f(Packed<4, EPI_LSTM_STEP, 8, 1, 1, 2>());
    if (K <= 256) return f(Packed<4, EPI_LSTM_STEP, 8, 2, 1, 2>());
    if (K <= 384) return f(Packed<4, EPI_LSTM_STEP, 8, 3, 1, 2>());
    return f(Packed<4, EPI_LSTM_STEP, 8, 4, 1, 2>());
  }
  if (variant == 0) return K <= 256 ? f(Packed<1, EPI_RNN_STEP, 4, 2, 1, 1>()) : f(Packed<1, EPI_RNN_STEP, 4, 4, 1, 1>());
  if (variant == 1) return K <= 256 ? f(Packed<2, EPI_RNN_STEP, 4, 2, 1, 1>()) : f(Packed<2, EPI_RNN_STEP, 4, 4, 1, 1>());
  if (variant == 2) return K <= 256 ? f(Packed<4, EPI_RNN_STEP, 4, 2, 1, 1>()) : f(Packed<4, EPI_RNN_STEP, 4, 4, 1, 1>());
  if (H % 64 == 0) return K <= 256 ? f(Packed<4, EPI_RNN_STEP, 8, 1, 2, 1>()) : f(Packed<4, EPI_RNN_STEP, 8, 2, 2, 1>());
  return K <= 256 ? f(Packed<2, EPI_RNN_STEP, 8, 1, 2, 1>()) : f(Packed<2, EPI_RNN_STEP, 8, 2, 2, 1>());
}

}  // namespace

int packed_members(CellEpilogue epi, int32_t H, int32_t variant) {
  if (epi == EPI_TREE_INTERNAL) return H / 16;
  if (epi == EPI_LSTM_STEP) return H / (variant == 0 ? 16 : 32);
  return H / (variant == 0 ? 16 : variant == 1 || H % 64 ? 32 : 64);
}

int packed_groups(CellEpilogue epi, int32_t H, int32_t K, int32_t variant, int32_t n_cu) {
  const bool tree = epi == EPI_TREE_INTERNAL;
  if ((!tree && epi != EPI_LSTM_STEP && epi != EPI_RNN_STEP) || K <= 0 || K > (tree ? kStationaryMaxK : kStationaryMaxStepK) ||
      H <= 0 || H % 32)
    return 0;
  int per_cu = dispatch(epi, H, K, variant, [](auto k) { return decltype(k)::per_cu(); });
  // a second workgroup on a compute unit only gets in the way of a recurrence's first
  if (!tree) per_cu = std::min(per_cu, 1);
  return 8 * std::min(per_cu * (n_cu / 8) / packed_members(epi, H, variant), kTreeMaxGroups / 8);
}

// A step takes a workgroup longer the more units it has, and the longer the more row blocks there are for a group: as few
// units as leave every group a single block of 16 rows, else the instances that multiply two blocks between two barriers, or
// two unit blocks.  Forward calls, us, sequences of 1 to 60 (LSTM) or 1 to 40 steps (BiRNN): LSTM H = 512, 128 sequences 212
// with 16 units and 236 with 32, 256 sequences 279 and 261; H = 256 174 and 190, 256 sequences 184 and 202, 400 sequences 223
// and 214; BiRNN H = 512, 128 sequences 158 with 32 units, 169 with 64, 176 with 64 and eight wavefronts, 256 sequences 217,
// 199 and 206, 900 sequences 560, 472 and 446.
int packed_variant(CellEpilogue epi, int32_t H, int32_t n_live, int32_t directions, int32_t n_cu) {
  if (epi == EPI_TREE_INTERNAL) return 0;
  const int last = epi == EPI_LSTM_STEP ? 1 : 3;
  for (int v = 0; v < last; ++v) {
    if (epi == EPI_RNN_STEP && v == 2 && H % 64) continue;
    if (n_live <= 16 * (packed_groups(epi, H, H, v, n_cu) / directions)) return v;
  }
  return last;
}

hipError_t launch_packed(CellEpilogue epi, const StationaryArgs& s, hipStream_t stream, const LaunchEvents& ev) {
  return dispatch(epi, s.a[0].H, s.a[0].nseg * s.a[0].kseg, s.variant, [&](auto k) { return decltype(k)::launch(s, stream, ev); });
}

hipError_t launch_pack_states(const PackStatesArgs& p, hipStream_t stream, const LaunchEvents& ev) {
  launch_with_events(pack_states_kernel, dim3((unsigned)((p.n + 3) / 4)), dim3(256), 0, stream, ev.start, ev.stop, p);
  return hipGetLastError();
}

}  // namespace acrobat
