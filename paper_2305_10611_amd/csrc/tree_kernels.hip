// Weight-stationary cell kernels for gfx950: a workgroup keeps the weight rows of 16 hidden units (all G gates) in
// its registers and node rows stream past them, 16 at a time.  They take small leaf levels and the tree levels whose
// operands do not arrive packed: level by level under capture, wide levels of a few large trees on the whole chip, calls
// without room for packed operands.  All levels in one launch otherwise run on packed_kernels.hip, with the same bits, and
// large leaf levels on dense_kernels.hip.
//
// What this is for.  The level kernels fetch weight tiles again for every node tile: 640 KB of weights per 64 nodes at
// H = 512, which is what bounds a level of a few hundred nodes, and every level of a tree batch is a launch of its own.
// Here the weights of a cell are spread over the register files of the H / 16 workgroups of a GROUP - at H = 512 the
// 32 compute units of one XCD hold all of U, 328 of their 512 KB of registers each - and the only operand that moves
// is node rows, out of that XCD's L2.  The trees of a batch are dealt out to the groups; a node needs rows of its own
// tree only, so a group runs all levels of its trees in ONE launch and its workgroups wait for each other between
// levels (arrival counter, write-through stores, agent-scope loads: the exchange of the persistent recurrences).
//
// Contraction.  fp16 matrix cores on split operands (split_fp16.h): weights are split once when they are loaded, node
// rows on their way into the operand registers.  Wavefront w of NW takes the 32-k steps w, w + NW, ... of the
// contraction for all G * 16 columns: v_mfma_f32_16x16x32_f16, lane l supplies A[row l % 16][k] and B[k][column l % 16]
// for k = 4 (l / 16) + 0 .. 3 and 16 more (two loads of 64 contiguous bytes per row and step) and holds
// z[row 4 (l / 16) + v][column l % 16] in result register v.  A step's registers are requested again for the next
// rows as soon as they have been split, so a block's rows are under way while the block before it is multiplied.
// The NW partial sums meet in LDS (two buffers, one barrier per block); with eight wavefronts the threads of one half
// finish even blocks and those of the other half odd ones, with four - two workgroups then share a compute unit - all
// threads finish.
//
// Bound: the chain of dependent steps.  A level of one block per group takes 3 us (stores complete, arrival counter, rows,
// 60 matrix instructions per wavefront, sums, gates), against 5 to 15 us for a launch of its own; a further block of 16
// rows 2.4 us at H = 512, of which 0.8 us are matrix instructions (operands packed: 1.8).  TreeLSTM forward, 256 trees, H
// = 512: 672 -> 317 us; 64 trees, H = 256: 143 -> 95 us (with the wide leaf levels on the split tiles; with packed
// operands and rows 247 and 68).  Tried: handing the buffers from wavefront to wavefront with counters in LDS instead of
// the barrier (117 instead of 99 us on 2 943 rows), a loop per turn so that the waits are exact (171 registers spilled).
#include "tree_kernels.h"

#include "cell_epilogue.h"
#include "packed_rows.h"
#include "split_fp16.h"

#include <algorithm>
#include <atomic>
#include <type_traits>

namespace acrobat {
namespace {

constexpr int kZRow = 20;  // padded row of partial sums: the four rows of a result register fall on different banks

// kStates: node rows are states, |h| <= 1, that other workgroups of the launch may have stored (agent-scope loads, one
// scale for all); else rows of an input matrix (plain loads, a scale for every row and wavefront).
constexpr int kListRows = 512;  // list positions of a level whose index lists sit in LDS at a time

template <int G, int EPI, int NW, int NS, int RB>
__global__ __launch_bounds__(64 * NW, 2) void cell_stationary_kernel(const StationaryArgs s) {
  constexpr bool kTree = EPI == EPI_TREE_INTERNAL, kStates = kTree;  // two operand rows per node, states
  constexpr int BR = 16 * RB;         // rows of a block
  constexpr int ZW = G * BR * kZRow;  // floats of one wavefront's partial sums: [gate][row][column]
  constexpr int TURNS = NW / 4;       // groups of 256 threads that take turns at finishing a block
  extern __shared__ __attribute__((aligned(16))) float zbuf[];  // [2][NW][ZW]
  __shared__ int l_out[2][kListRows], l_r0[2][kListRows], l_r1[kTree ? 2 : 1][kTree ? kListRows : 1];  // row written, operand rows
  __shared__ float s_bias[G][16], s_winv[NW][G][16];
  __shared__ int s_go;

  // workgroup ids that agree modulo 8 share an XCD (placement only matters for speed)
  const int slot = blockIdx.x >> 3;
  const int group = (slot / s.n_cb) * 8 + (blockIdx.x & 7), cb = slot % s.n_cb;
  if (group >= s.n_groups) return;
  const CellLevelArgs& a = s.a[s.two ? group & 1 : 0];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, kq = lane >> 4;
  const int H = a.H, T = (a.nseg * a.kseg) >> 5;  // 32-k steps, at most NW * NS

  // ---- this wavefront's weights: gate g, unit 16 cb + li, steps w + NW t
  half8 whi[G][NS], wlo[G][NS];
  {
    floatx4 raw[G][NS][2];  // (every load in flight at once)
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const float* row = a.W + ((size_t)gate_row<EPI>(g) * H + 16 * cb + li) * (size_t)a.ldw + 4 * kq;
#pragma unroll
      for (int t = 0; t < NS; ++t) {
        const int step = w + NW * t;
        raw[g][t][0] = raw[g][t][1] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        if (step < T) {
          raw[g][t][0] = *reinterpret_cast<const floatx4*>(row + 32 * step);
          raw[g][t][1] = *reinterpret_cast<const floatx4*>(row + 32 * step + 16);
        }
      }
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      float m = 0.0f;
#pragma unroll
      for (int t = 0; t < NS; ++t) m = largest(raw[g][t][1], largest(raw[g][t][0], m));
      const float sc = scale_for(largest_of_quarters(m));
      if (lane < 16) {
        const float unit = inverse_power(sc) * (kStates ? 1.0f / kStateScale : 1.0f);
        s_winv[w][g][li] = kStates && unit > kLargestUnit ? __builtin_inff() : unit;  // (the sums are not finite then)
      }
      if (w == 0 && lane < 16) s_bias[g][li] = a.bias ? a.bias[gate_row<EPI>(g) * H + 16 * cb + li] : 0.0f;
#pragma unroll
      for (int t = 0; t < NS; ++t) split8(raw[g][t][0], raw[g][t][1], sc, whi[g][t], wlo[g][t]);
    }
  }

  // ---- node rows: a ring of the NS steps of one block.  Steps past the contraction range and rows past the last block
  // are requested past the end of the buffer, which reads zeros: no branch between the matrix instructions.
  const __amdgpu_buffer_rsrc_t rsrc = agent_buffer(a.src0, s.src_bytes);
  const int steps0 = a.kseg >> 5;  // steps of the first segment
  const __amdgpu_buffer_rsrc_t places = agent_buffer(s.operand, s.operand ? s.operand_bytes : 0u);  // leaves only
  floatx4 ring[RB][NS][2];
  unsigned base0[RB], base1[RB];     // byte offset of this lane's part of its row at step 0 (second segment: less kseg)
  auto request = [&](int r, int t, bool more) {
    const int step = w + NW * t;
    unsigned at = (kTree && step >= steps0 ? base1[r] : base0[r]) + 128u * step;
    at = more && step < T ? at : 0xffffff00u;
    if constexpr (kStates) {
      ring[r][t][0] = load_agent_f4(rsrc, at);
      ring[r][t][1] = load_agent_f4(rsrc, at + 64u);
    } else {
      ring[r][t][0] = load_buffer_f4(rsrc, at);
      ring[r][t][1] = load_buffer_f4(rsrc, at + 64u);
    }
  };

  // the elements this thread finishes in its turn: rows er, er + 16, ... of the block, unit j
  const int turn = TURNS == 2 ? w >> 2 : 0;
  const int er = (tid & 255) >> 4, eu = tid & 15, j = 16 * cb + eu;
  unsigned* const counter = s.counters + (size_t)group * kTreeCounterStride;
  unsigned arrived = 0;  // levels this group has announced

  // The group's share of a level: positions [p0, p1) of the lists, in chunks of kListRows whose index lists sit in LDS
  // (two buffers: the next chunk's lists are fetched while the stores of this one complete).
  auto share_of = [&](int lv, int& p0, int& p1) {
    if (s.off) {
      p0 = s.off[lv * s.n_groups + group];
      p1 = s.off[lv * s.n_groups + group + 1];
    } else {  // an even share of all rows, in whole blocks
      const int blocks = (a.n + BR - 1) / BR;
      p0 = BR * (int)((long)blocks * group / s.n_groups);
      p1 = BR * (int)((long)blocks * (group + 1) / s.n_groups);
      p1 = p1 < a.n ? p1 : a.n;
    }
  };
  constexpr int PE = kListRows / (64 * NW);
  int list_out[PE], list_r0[PE], list_r1[PE];
  auto request_lists = [&](int p0, int p1) {  // tail rows repeat the last node; never stored
#pragma unroll
    for (int e = 0; e < PE; ++e) {
      int p = p0 + tid + 64 * NW * e;
      p = p < p1 ? p : p1 - 1;
      list_out[e] = a.out_rows ? a.out_rows[p] : p;
      list_r0[e] = a.idx0 ? a.idx0[p] : p;
      list_r1[e] = kTree ? a.idx1[p] : 0;
    }
  };
  auto keep_lists = [&](int buf) {
#pragma unroll
    for (int e = 0; e < PE; ++e) {
      l_out[buf][tid + 64 * NW * e] = list_out[e];
      l_r0[buf][tid + 64 * NW * e] = list_r0[e];
      if constexpr (kTree) l_r1[buf][tid + 64 * NW * e] = list_r1[e];
    }
  };
  int lv = s.level0, p0, p1, lists = 0;
  share_of(lv, p0, p1);
  if (p0 >= p1) return;  // (nothing in this level: nothing in a later one)
  request_lists(p0, p1);
  keep_lists(0);
  int q0 = 0, q1 = 0;  // the share of the next level
  if (lv + 1 < s.level1) share_of(lv + 1, q0, q1);
  __syncthreads();
  for (bool new_level = true;; lists ^= 1) {
    const int n = p1 - p0 < kListRows ? p1 - p0 : kListRows, nb = (n + BR - 1) / BR;
    const int* const s_out = l_out[lists];
    const int* const s_r0 = l_r0[lists];
    const int* const s_r1 = l_r1[kTree ? lists : 0];
    // What comes next: the rest of this level, the next level, or nothing (a group's levels only get narrower).  Lists and
    // offsets are cold - nobody has read them yet - so they are requested one and two levels ahead, behind the level's own
    // loads, which would otherwise wait for them (loads return in order).
    const bool last_chunk = p0 + kListRows >= p1;
    const int c0 = last_chunk ? __builtin_amdgcn_readfirstlane(q0) : p0 + kListRows;
    const int c1 = last_chunk ? __builtin_amdgcn_readfirstlane(q1) : p1;
    int n0 = 0, n1 = 0;
    EpilogueOperands<G, EPI, RB> eo;
    auto fetch_operands = [&](int b) {  // of the gate arithmetic; rows of this workgroup's own units and inputs only
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        const int i = BR * b + 16 * r + er;
        eo.live[r] = i < n;
        eo.orow[r] = (size_t)s_out[i];
        if constexpr (EPI == EPI_TREE_INTERNAL) {
          eo.p0[r] = a.cprev_src[(size_t)s_r0[i] * H + j];
          eo.p1[r] = a.cprev_src[(size_t)s_r1[i] * H + j];
        }
      }
    };
    if (new_level && arrived > 0) {  // the group's previous level is complete once all its workgroups have announced it
      if (tid == 0) s_go = wait_for(counter, (unsigned)s.n_cb * arrived, s.status, s.max_polls) ? 1 : 0;
      __syncthreads();
      if (!s_go) break;
    }
    {
      auto set_rows = [&](int b) {
#pragma unroll
        for (int r = 0; r < RB; ++r) {
          const int i = BR * b + 16 * r + li;
          base0[r] = (unsigned)s_r0[i] * (unsigned)a.ld0 * 4u + 16u * kq;
          if constexpr (kTree) base1[r] = (unsigned)s_r1[i] * (unsigned)a.ld0 * 4u + 16u * kq - 128u * steps0;
        }
      };
      set_rows(0);
#pragma unroll
      for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int t = 0; t < NS; ++t) request(r, t, true);
      set_rows(nb > 1 ? 1 : 0);
      if (turn == 0) fetch_operands(0);
      if (c0 < c1) request_lists(c0, c1);
      if (last_chunk && lv + 2 < s.level1) share_of(lv + 2, n0, n1);

      for (int b = 0; b < nb; ++b) {
        const bool mine = TURNS == 1 || (b & 1) == turn;
        const bool more = b + 1 < nb;
        if (mine && b > 0) fetch_operands(b);
        float* const z = zbuf + (b & 1) * (NW * ZW) + w * ZW;
#pragma unroll
        for (int r = 0; r < RB; ++r) {
          float sc = kStateScale, inv[4];
          if constexpr (!kStates) {
            float m = 0.0f;
#pragma unroll
            for (int t = 0; t < NS; ++t) m = largest(ring[r][t][1], largest(ring[r][t][0], m));
            sc = scale_for(largest_of_quarters(m));
            const float rinv = inverse_power(sc);
#pragma unroll
            for (int v = 0; v < 4; ++v) inv[v] = __shfl(rinv, 4 * kq + v);  // (lane i < 16 holds row i)
          }
          floatx4 acc[G];
#pragma unroll
          for (int g = 0; g < G; ++g) acc[g] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int t = 0; t < NS; ++t) {
            half8 ahi, alo;
            split8(ring[r][t][0], ring[r][t][1], sc, ahi, alo);
            request(r, t, more);
#pragma unroll
            for (int g = 0; g < G; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(alo, whi[g][t], acc[g], 0, 0, 0);
#pragma unroll
            for (int g = 0; g < G; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ahi, wlo[g][t], acc[g], 0, 0, 0);
#pragma unroll
            for (int g = 0; g < G; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ahi, whi[g][t], acc[g], 0, 0, 0);
          }
#pragma unroll
          for (int g = 0; g < G; ++g) {
            const float winv = s_winv[w][g][li];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              float unit = winv;
              if constexpr (!kStates) {
                unit *= inv[v];
                unit = unit > kLargestUnit ? __builtin_inff() : unit;
              }
              z[(g * BR + 16 * r + 4 * kq + v) * kZRow + li] = acc[g][v] * unit;
            }
          }
        }
        set_rows(b + 2 < nb ? b + 2 : 0);
        // (a buffer written two blocks ago has been read: its readers have passed the barrier in between)
        __syncthreads();
        if (mine) {
          const float* const zr = zbuf + (b & 1) * (NW * ZW);  // (what this thread adds up nobody else reads)
          float zs[G][RB];
          float finite = 0.0f;
          auto sum_up = [&]() {
#pragma unroll
            for (int g = 0; g < G; ++g) {
              eo.bz[g] = s_bias[g][eu];
#pragma unroll
              for (int r = 0; r < RB; ++r) {
                float sum = 0.0f;
#pragma unroll
                for (int q = 0; q < NW; ++q) sum += zr[q * ZW + (g * BR + 16 * r + er) * kZRow + eu];
                zs[g][r] = sum;
                finite = __builtin_fmaf(sum, 0.0f, finite);
              }
            }
          };
          sum_up();
          if (__builtin_expect(finite != 0.0f, 0)) {
            // What is not finite, or not to be split, is computed in fp32.  (The result takes the place of the first
            // partial sum in LDS, which only this thread reads: kept in registers, it would cost spills in every block.)
            float* const zw = zbuf + (b & 1) * (NW * ZW);
#pragma unroll 1
            for (int e = 0; e < G * RB; ++e) {
              const int g = e / RB, row = 16 * (e % RB) + er;
              float sum = 0.0f;
#pragma unroll 1
              for (int q = 0; q < NW; ++q) sum += zw[q * ZW + (g * BR + row) * kZRow + eu];
              if (__builtin_isfinite(sum)) continue;
              const float* const wr = a.W + ((size_t)gate_row<EPI>(g) * H + j) * (size_t)a.ldw;
              const unsigned at0 = (unsigned)s_r0[BR * b + row] * (unsigned)a.ld0 * 4u;
              const unsigned at1 = kTree ? (unsigned)s_r1[BR * b + row] * (unsigned)a.ld0 * 4u - 4u * a.kseg : at0;
              sum = 0.0f;
#pragma unroll 1
              for (int k = 0; k < 32 * T; k += 4) {
                const unsigned at = (k < a.kseg ? at0 : at1) + 4u * k;
                floatx4 x;
                if constexpr (kStates) x = load_agent_f4(rsrc, at);
                else x = load_buffer_f4(rsrc, at);
                const floatx4 wk = *reinterpret_cast<const floatx4*>(wr + k);
#pragma unroll
                for (int c = 0; c < 4; ++c) sum = __builtin_fmaf(x[c], wk[c], sum);
              }
#pragma unroll 1
              for (int q = 1; q < NW; ++q) zw[q * ZW + (g * BR + row) * kZRow + eu] = 0.0f;
              zw[(g * BR + row) * kZRow + eu] = sum;
            }
            sum_up();
          }
          epilogue_apply<G, EPI, RB, kStates>(a, j, [&](int g, int r) { return zs[g][r]; }, eo, [&](int r, float h, float c) {
            if (EPI == EPI_TREE_LEAF && s.operand)
              store_tree_place(places, s.cells, H, s.place[p0 + BR * b + 16 * r + er], cb, eu, lane, h, c);
          });
        }
      }
    }
    if (c0 < c1) keep_lists(lists ^ 1);
    if (last_chunk && s.stamps && cb == 0 && tid == 0) s.stamps[lv * s.n_groups + group] = wall_clock64();
    const bool announce = last_chunk && lv + 1 < s.level1;
    if (announce) wait_stores_done();  // this wavefront's stores have completed ...
    __syncthreads();                   // ... and so have the other wavefronts'; the lists are complete
    if (announce) {
      if (tid == 0) __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      ++arrived;
    }
    if (c0 >= c1) break;
    p0 = c0;
    p1 = c1;
    new_level = last_chunk;
    if (last_chunk) {
      ++lv;
      q0 = n0;
      q1 = n1;
    }
  }
  if (arrived > 0 && tid == 0) leave_block(counter, s.n_cb);
}

// One narrow tree level as a launch of its own, for calls that may not use launches that wait (captured ones): the kernel
// above would fetch whole weights for a block or two of rows, 328 KB per compute unit at H = 512, 6.5 us.  Here
// every wavefront of it is a workgroup: part q of NW fetches 1 / NW of the weights, multiplies its share of the contraction
// and leaves the partial sums in memory (write-through stores, then a ticket); the wavefront that draws the last ticket of a
// block adds the parts up in the order of the kernel above and finishes the block.  Nobody waits, and every sum is rounded
// as there, so the results are the same bit for bit.
// Bound: the launch, 1 / NW of the weights at 50 KB/us per compute unit, and the exchange.  Captured calls replay in, 8
// trees of 20 leaves, H = 512 175 -> 116 us, H = 256 100 -> 86, 256 trees, H = 512 556 -> 501.
template <int NW, int NS>
__global__ __launch_bounds__(64) void cell_parts_kernel(const StationaryArgs s, const int p_first, const int n, float* const partial,
                                                       unsigned* const tickets) {
  constexpr int G = 5, EPI = EPI_TREE_INTERNAL;
  constexpr int kPartFloats = G * 256;  // [gate][column][row]
  const CellLevelArgs& a = s.a[0];
  const int q = blockIdx.x % NW, cb = blockIdx.x / NW, b = blockIdx.y;
  const int lane = threadIdx.x, li = lane & 15, kq = lane >> 4;
  const int H = a.H, T = (a.nseg * a.kseg) >> 5, j = 16 * cb + li;

  // this lane's operand row, its part of the steps q + NW t
  const auto position = [&](int i) { return p_first + (16 * b + i < n ? 16 * b + i : n - 1); };  // tail rows repeat the last node
  const int pl = position(li), steps0 = a.kseg >> 5;
  const unsigned base0 = (unsigned)(a.idx0 ? a.idx0[pl] : pl) * (unsigned)a.ld0 * 4u + 16u * kq;
  const unsigned base1 = (unsigned)a.idx1[pl] * (unsigned)a.ld0 * 4u + 16u * kq - 128u * steps0;
  const __amdgpu_buffer_rsrc_t rsrc = agent_buffer(a.src0, s.src_bytes);
  // (what the gates need is requested by every part: the one that finishes would wait for it twice, lists and rows)
  EpilogueOperands<G, EPI, 4> eo;
  int r0[4], r1[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int p = position(4 * kq + v);
    eo.live[v] = 16 * b + 4 * kq + v < n;
    eo.orow[v] = (size_t)(a.out_rows ? a.out_rows[p] : p);
    r0[v] = a.idx0 ? a.idx0[p] : p;
    r1[v] = a.idx1[p];
  }
  floatx4 raw[G][NS][2], x[NS][2];
#pragma unroll
  for (int t = 0; t < NS; ++t) {
    const int step = q + NW * t;
    unsigned at = (step >= steps0 ? base1 : base0) + 128u * step;
    at = step < T ? at : 0xffffff00u;
    x[t][0] = load_buffer_f4(rsrc, at);
    x[t][1] = load_buffer_f4(rsrc, at + 64u);
  }
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const float* row = a.W + ((size_t)gate_row<EPI>(g) * H + j) * (size_t)a.ldw + 4 * kq;
#pragma unroll
    for (int t = 0; t < NS; ++t) {
      const int step = q + NW * t;
      raw[g][t][0] = raw[g][t][1] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
      if (step < T) {
        raw[g][t][0] = *reinterpret_cast<const floatx4*>(row + 32 * step);
        raw[g][t][1] = *reinterpret_cast<const floatx4*>(row + 32 * step + 16);
      }
    }
  }
  half8 whi[G][NS], wlo[G][NS];
  float unit[G];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    float m = 0.0f;
#pragma unroll
    for (int t = 0; t < NS; ++t) m = largest(raw[g][t][1], largest(raw[g][t][0], m));
    const float sc = scale_for(largest_of_quarters(m));
    unit[g] = inverse_power(sc) * (1.0f / kStateScale);
    if (unit[g] > kLargestUnit) unit[g] = __builtin_inff();
#pragma unroll
    for (int t = 0; t < NS; ++t) split8(raw[g][t][0], raw[g][t][1], sc, whi[g][t], wlo[g][t]);
  }
  floatx4 acc[G];
#pragma unroll
  for (int g = 0; g < G; ++g) acc[g] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int t = 0; t < NS; ++t) {
    half8 ahi, alo;
    split8(x[t][0], x[t][1], kStateScale, ahi, alo);
#pragma unroll
    for (int g = 0; g < G; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(alo, whi[g][t], acc[g], 0, 0, 0);
#pragma unroll
    for (int g = 0; g < G; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ahi, wlo[g][t], acc[g], 0, 0, 0);
#pragma unroll
    for (int g = 0; g < G; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ahi, whi[g][t], acc[g], 0, 0, 0);
  }

  // rows 4 kq + v of column li, part q
  const size_t block = (size_t)b * s.n_cb + cb;
  const __amdgpu_buffer_rsrc_t parts = agent_buffer(partial + block * (NW * kPartFloats), NW * kPartFloats * sizeof(float));
  const unsigned at = 4u * (16 * li + 4 * kq);
#pragma unroll
  for (int g = 0; g < G; ++g) {
    floatx4 z;
#pragma unroll
    for (int v = 0; v < 4; ++v) z[v] = acc[g][v] * unit[g];
    store_agent_f4(parts, (unsigned)(q * kPartFloats + g * 256) * 4u + at, z);
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    eo.p0[v] = a.cprev_src[(size_t)r0[v] * H + j];
    eo.p1[v] = a.cprev_src[(size_t)r1[v] * H + j];
  }
#pragma unroll
  for (int g = 0; g < G; ++g) eo.bz[g] = a.bias ? a.bias[gate_row<EPI>(g) * H + j] : 0.0f;
  wait_stores_done();
  unsigned drawn = 0;
  if (lane == 0) drawn = __hip_atomic_fetch_add(tickets + block, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (__builtin_amdgcn_readfirstlane((int)drawn) != NW - 1) return;
  if (lane == 0) __hip_atomic_store(tickets + block, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

  float zs[G][4], finite = 0.0f;
#pragma unroll
  for (int g = 0; g < G; ++g) {
    floatx4 part[NW];
#pragma unroll
    for (int e = 0; e < NW; ++e) part[e] = load_agent_f4(parts, (unsigned)(e * kPartFloats + g * 256) * 4u + at);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      float sum = 0.0f;
#pragma unroll
      for (int e = 0; e < NW; ++e) sum += part[e][v];
      zs[g][v] = sum;
      finite = __builtin_fmaf(sum, 0.0f, finite);
    }
  }
  if (__builtin_expect(finite != 0.0f, 0)) {  // in fp32, as above
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if (__builtin_isfinite(zs[g][v])) continue;
        const float* const wr = a.W + ((size_t)gate_row<EPI>(g) * H + j) * (size_t)a.ldw;
        const unsigned at0 = (unsigned)r0[v] * (unsigned)a.ld0 * 4u;
        const unsigned at1 = (unsigned)r1[v] * (unsigned)a.ld0 * 4u - 4u * a.kseg;
        float sum = 0.0f;
#pragma unroll 1
        for (int k = 0; k < 32 * T; k += 4) {
          const floatx4 xk = load_buffer_f4(rsrc, (k < a.kseg ? at0 : at1) + 4u * k);
          const floatx4 wk = *reinterpret_cast<const floatx4*>(wr + k);
#pragma unroll
          for (int c = 0; c < 4; ++c) sum = __builtin_fmaf(xk[c], wk[c], sum);
        }
        zs[g][v] = sum;
      }
  }
  epilogue_apply<G, EPI, 4>(a, j, [&](int g, int v) { return zs[g][v]; }, eo);
}

template <int G, int EPI, int NW, int NS>
struct Stationary {
  // 16-row blocks multiplied between two barriers: the states of many gates leave no registers for a second one
  static constexpr int RB = EPI == EPI_TREE_INTERNAL ? 1 : 2;
  static constexpr size_t kLdsBytes = (size_t)2 * NW * G * 16 * RB * kZRow * sizeof(float);
  static const void* kernel() { return reinterpret_cast<const void*>(&cell_stationary_kernel<G, EPI, NW, NS, RB>); }
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
    launch_with_events((cell_stationary_kernel<G, EPI, NW, NS, RB>), dim3(grid), dim3(64 * NW), kLdsBytes, stream, ev.start, ev.stop, s);
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

// Calls f with the Stationary of the smallest instance that holds K columns: four wavefronts (two workgroups per
// compute unit) up to K = 512, eight up to 1 024.
template <int G, int EPI, class F>
auto dispatch_steps(int32_t K, F&& f) {
  if (K <= 128) return f(Stationary<G, EPI, 4, 1>());
  if (K <= 256) return f(Stationary<G, EPI, 4, 2>());
  if (K > 768) return f(Stationary<G, EPI, 8, 4>());
  if (K > 512) return f(Stationary<G, EPI, 8, 3>());
  return f(Stationary<G, EPI, 4, 4>());
}
template <class F>
auto dispatch(CellEpilogue epi, int32_t K, F&& f) {
  return epi == EPI_TREE_LEAF ? dispatch_steps<3, EPI_TREE_LEAF>(K, f) : dispatch_steps<5, EPI_TREE_INTERNAL>(K, f);
}

}  // namespace

int stationary_groups(CellEpilogue epi, int32_t H, int32_t K, int32_t n_cu) {
  if ((epi != EPI_TREE_LEAF && epi != EPI_TREE_INTERNAL) || K <= 0 || K > kStationaryMaxK || H <= 0 || H % 16) return 0;
  const int per_xcd = dispatch(epi, K, [](auto k) { return decltype(k)::per_cu(); }) * (n_cu / 8);
  return 8 * std::min(per_xcd / (H / 16), kTreeMaxGroups / 8);
}

hipError_t launch_stationary(CellEpilogue epi, const StationaryArgs& s, hipStream_t stream, const LaunchEvents& ev) {
  return dispatch(epi, s.a[0].nseg * s.a[0].kseg, [&](auto k) { return decltype(k)::launch(s, stream, ev); });
}

hipError_t launch_tree_level(const StationaryArgs& s, int32_t p_first, int32_t n, const SplitKWorkspace& ws, hipStream_t stream,
                             const LaunchEvents& ev) {
  const int32_t K = s.a[0].nseg * s.a[0].kseg;
  const auto parts = [&](auto kernel, int nw) {
    const size_t blocks = (size_t)(n + 15) / 16, tickets = blocks * s.n_cb;
    if (tickets * nw * 5 * 256 > ws.partial_floats || tickets > (size_t)ws.n_counters) return false;
    launch_with_events(kernel, dim3((unsigned)(s.n_cb * nw), (unsigned)blocks), dim3(64), 0, stream, ev.start, ev.stop, s, p_first, n,
                       ws.partial, ws.counters);
    return true;
  };
  // (H = 64, weights of 41 KB: a stationary launch per level is as fast, 57 against 59 us for 8 trees)
  if (n <= kPartsMaxRows && K > 128 &&
      (K <= 256 ? parts(cell_parts_kernel<4, 2>, 4) : K <= 512 ? parts(cell_parts_kernel<4, 4>, 4) :
       K <= 768 ? parts(cell_parts_kernel<8, 3>, 8) : parts(cell_parts_kernel<8, 4>, 8)))
    return hipGetLastError();
  return launch_stationary(EPI_TREE_INTERNAL, s, stream, ev);
}

}  // namespace acrobat
