// What every cell kernel shares: constants, gate functions and the fused epilogue (device code, gfx950).
#pragma once
#include "cell_kernels.h"

#include "agent_access.h"

namespace acrobat {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kBK = 32;        // k columns per slab
constexpr int kThreads = 256;
constexpr int kBlockFloats = 16 * 64;  // one 32x32 accumulator block of one wavefront

// The kernels for small levels number their workgroups (node tile, unit tile) with the unit tile fastest and pad
// the number of unit tiles to a multiple of 8: workgroup ids go round-robin to the 8 XCDs, so every node tile of a
// unit tile then runs on the same XCD and finds that tile's weight rows in its L2.  With fewer than 8 unit tiles
// the padding would leave XCDs empty, so there is none.
__host__ __device__ constexpr int padded_unit_tiles(int n_jt) { return n_jt >= 8 ? (n_jt + 7) & ~7 : n_jt; }

__device__ __forceinline__ float fast_sigmoid(float x) {
  return __builtin_amdgcn_rcpf(1.0f + __expf(-x));  // exp -> inf gives 0, exp -> 0 gives 1
}
__device__ __forceinline__ float fast_tanh(float x) {
  return 1.0f - 2.0f * __builtin_amdgcn_rcpf(__expf(2.0f * x) + 1.0f);  // saturates to +-1
}

template <int EPI>
__device__ __forceinline__ constexpr int gate_row(int g) {
  // row block (in units of H) of computed gate g inside the weight matrix
  return EPI == EPI_TREE_LEAF ? (g == 0 ? 0 : g + 2) : g;  // leaf: i, o, u = blocks 0, 3, 4
}

// Fused epilogue of one lane: bias, gates, state update, scatter to the arena, for NV
// accumulator rows (node_of(v)) of hidden unit j; acc(g, v) is the pre-activation of gate g.
// Two stages.  epilogue_fetch reads the indices and then every gathered operand (all loads of a
// pass in flight together instead of one dependent chain per row); it depends on nothing the
// contraction computes, so a kernel may run it ahead of its k loop.  epilogue_apply does the
// arithmetic and the stores (the stores may alias the loads as far as the compiler can tell,
// which would otherwise serialise the rows).
//
// `sidx` (may be null) is the tile's index table in LDS, [3][bm]: arena row written, first and
// second operand row of tile row r = node - m0, as staged by the contraction kernel's prologue
// (tail rows hold the entries of node n - 1); without it the indices come from global memory.
template <int G, int EPI, int NV>
struct EpilogueOperands {
  float bz[G];
  size_t orow[NV];
  bool live[NV];
  float p0[NV], p1[NV];                        // gathered state: c of the two children / previous c / hoisted z (RNN)
  float zx[EPI == EPI_LSTM_STEP ? G : 1][NV];  // hoisted input transform of an LSTM step
};

template <int G, int EPI, int NV, class NodeOf>
__device__ __forceinline__ void epilogue_fetch(const CellLevelArgs& a, const int j, NodeOf&& node_of,
                                               EpilogueOperands<G, EPI, NV>& o, const int* sidx = nullptr, const int bm = 0,
                                               const int m0 = 0) {
  const int H = a.H, n = a.n;
#pragma unroll
  for (int g = 0; g < G; ++g) {
    if constexpr (EPI == EPI_RELU_OUT) o.bz[g] = a.bias && j < a.n_cols ? a.bias[j] : 0.0f;
    else o.bz[g] = a.bias ? a.bias[gate_row<EPI>(g) * H + j] : 0.0f;
  }
  int ia[NV], ib[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int node = node_of(v);
    o.live[v] = node < n;
    const int nd = o.live[v] ? node : n - 1;  // tail rows read what the last node reads, store nothing
    ia[v] = ib[v] = 0;
    if (sidx) {
      const int r = node - m0;
      o.orow[v] = (size_t)sidx[r];
      if constexpr (EPI == EPI_TREE_INTERNAL || EPI == EPI_LSTM_STEP) ia[v] = sidx[bm + r];
      if constexpr (EPI == EPI_TREE_INTERNAL) ib[v] = sidx[2 * bm + r];
    } else {
      o.orow[v] = a.out_rows ? (size_t)a.out_rows[nd] : (size_t)nd;
      if constexpr (EPI == EPI_TREE_INTERNAL) {
        ia[v] = a.idx0[nd];
        ib[v] = a.idx1[nd];
      }
      if constexpr (EPI == EPI_LSTM_STEP) {
        if (a.cprev_src) ia[v] = a.idx0[nd];
      }
    }
  }
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    o.p0[v] = o.p1[v] = 0.0f;
    if constexpr (EPI == EPI_TREE_INTERNAL) {
      o.p0[v] = a.cprev_src[(size_t)ia[v] * H + j];
      o.p1[v] = a.cprev_src[(size_t)ib[v] * H + j];
    } else if constexpr (EPI == EPI_RNN_STEP) {
      o.p0[v] = a.zadd ? a.zadd[o.orow[v] * (size_t)H + j] : 0.0f;
    } else if constexpr (EPI == EPI_LSTM_STEP) {
      o.p0[v] = a.cprev_src ? a.cprev_src[(size_t)ia[v] * H + j] : 0.0f;
#pragma unroll
      for (int g = 0; g < G; ++g) o.zx[g][v] = a.zadd[o.orow[v] * (size_t)(G * H) + g * H + j];
    }
  }
}

// kShared: h is read by other workgroups of the same launch, so it is stored at agent scope.
template <bool kShared>
__device__ __forceinline__ void store_h(float* p, float v) {
  if constexpr (kShared) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *p = v;
}

struct NoFurtherStates {
  __device__ __forceinline__ void operator()(int, float, float) const {}
};
// `further` gets a leaf's states (row v, h, c) as well.
template <int G, int EPI, int NV, bool kShared = false, class Acc, class Further = NoFurtherStates>
__device__ __forceinline__ void epilogue_apply(const CellLevelArgs& a, const int j, Acc&& acc,
                                               const EpilogueOperands<G, EPI, NV>& o, Further&& further = Further()) {
  const int H = a.H;
  const float* bz = o.bz;
  if constexpr (EPI == EPI_STORE_Z) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      if (!o.live[v]) continue;
#pragma unroll
      for (int g = 0; g < G; ++g) a.zout[o.orow[v] * (size_t)(G * H) + g * H + j] = acc(g, v) + bz[g];
    }
  } else if constexpr (EPI == EPI_TREE_LEAF) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      if (!o.live[v]) continue;
      const float c = fast_sigmoid(acc(0, v) + bz[0]) * fast_tanh(acc(2, v) + bz[2]);
      const float h = fast_sigmoid(acc(1, v) + bz[1]) * fast_tanh(c);
      a.c[o.orow[v] * H + j] = c;
      store_h<kShared>(a.h + o.orow[v] * H + j, h);
      further(v, h, c);
    }
  } else if constexpr (EPI == EPI_TREE_INTERNAL) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      if (!o.live[v]) continue;
      const float c = fast_sigmoid(acc(0, v) + bz[0]) * fast_tanh(acc(4, v) + bz[4]) +
                      fast_sigmoid(acc(1, v) + bz[1]) * o.p0[v] + fast_sigmoid(acc(2, v) + bz[2]) * o.p1[v];
      a.c[o.orow[v] * H + j] = c;
      store_h<kShared>(a.h + o.orow[v] * H + j, fast_sigmoid(acc(3, v) + bz[3]) * fast_tanh(c));
    }
  } else if constexpr (EPI == EPI_RNN_STEP) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      if (!o.live[v]) continue;
      store_h<kShared>(a.h + o.orow[v] * H + j, fast_sigmoid(acc(0, v) + o.p0[v] + bz[0]));
    }
  } else if constexpr (EPI == EPI_RELU_OUT) {
    if (j < a.n_cols) {
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        if (!o.live[v]) continue;
        a.y[o.orow[v] * (size_t)a.ldo + j] = fmaxf(acc(0, v) + bz[0], 0.0f);
      }
    }
  } else {  // EPI_LSTM_STEP
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      if (!o.live[v]) continue;
      const float c = fast_sigmoid(acc(1, v) + o.zx[1][v] + bz[1]) * o.p0[v] +
                      fast_sigmoid(acc(0, v) + o.zx[0][v] + bz[0]) * fast_tanh(acc(3, v) + o.zx[3][v] + bz[3]);
      a.c[o.orow[v] * H + j] = c;
      store_h<kShared>(a.h + o.orow[v] * H + j, fast_sigmoid(acc(2, v) + o.zx[2][v] + bz[2]) * fast_tanh(c));
    }
  }
}

template <int G, int EPI, int NV, class Acc, class NodeOf>
__device__ __forceinline__ void cell_epilogue(const CellLevelArgs& a, const int j, Acc&& acc, NodeOf&& node_of,
                                              const int* sidx = nullptr, const int bm = 0, const int m0 = 0) {
  EpilogueOperands<G, EPI, NV> o;
  epilogue_fetch<G, EPI, NV>(a, j, node_of, o, sidx, bm, m0);
  epilogue_apply<G, EPI, NV>(a, j, acc, o);
}

// accumulator rows a lane owns after the reduction over the WK wavefronts of a node block
template <int WK>
constexpr int kOwnedRows = 4 * (4 / WK);

// Sums the accumulators of the WK wavefronts that share a node block (floats needed in `smem`: WM * (WK - 1) * G *
// kBlockFloats); own[g][v] is this wavefront's share of the result, accumulator row tile_acc_row(wk, v).
template <int G, int WM, int WK>
__device__ __forceinline__ void reduce_k_waves(const floatx16 (&acc)[G], float* const smem, float (&own)[G][kOwnedRows<WK>]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave % WM, wk = wave / WM;
  // The WK wavefronts of a node block hold partial sums over their share of k.  They are added
  // by a reduce-scatter through LDS: wavefront wk ends up with the complete sums of the QPW = 4/WK
  // accumulator quads v4 = wk*QPW .. wk*QPW + QPW-1 (8 nodes each) and every wavefront runs the
  // epilogue for the rows it owns, so the gate arithmetic is spread over all four SIMDs.  Each
  // quad is summed in ascending wk order, whoever owns it.
  constexpr int QPW = 4 / WK;  // quads owned per wavefront
  if constexpr (WK == 1) {
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int v = 0; v < 16; ++v) own[g][v] = acc[g][v];
  } else {
    // inbox of wavefront (wm, o): (WK-1) senders x G gates x QPW quads, one float4 per lane each
    floatx4* red = reinterpret_cast<floatx4*>(smem);
    auto inbox = [&](int o, int sender, int g, int qi) {
      const int slot = sender < o ? sender : sender - 1;
      return ((((wm * WK + o) * (WK - 1) + slot) * G + g) * QPW + qi) * 64 + lane;
    };
    __syncthreads();
#pragma unroll
    for (int v4 = 0; v4 < 4; ++v4) {
      const int o = v4 / QPW, qi = v4 % QPW;
      if (o != wk) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
          floatx4 q;
#pragma unroll
          for (int e = 0; e < 4; ++e) q[e] = acc[g][v4 * 4 + e];
          red[inbox(o, wk, g, qi)] = q;
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int qi = 0; qi < QPW; ++qi) {
        floatx4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int src = 0; src < WK; ++src) {  // ascending wk, own contribution in its place
          floatx4 q;
          if (src == wk) {
#pragma unroll
            for (int o = 0; o < WK; ++o)
              if (o == wk) {
#pragma unroll
                for (int e = 0; e < 4; ++e) q[e] = acc[g][(o * QPW + qi) * 4 + e];
              }
          } else {
            q = red[inbox(wk, src, g, qi)];
          }
          sum += q;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) own[g][qi * 4 + e] = sum[e];
      }
  }
}

// accumulator row of a lane's owned row v: quad wk * QPW + v / 4, element v % 4
template <int WK>
__device__ __forceinline__ int tile_acc_row(int wk, int v) { return (wk * (4 / WK) + (v >> 2)) * 4 + (v & 3); }

// fused epilogue of a contracted tile (accumulator row r of a lane: node = m0 + 32 wm + 8 (r / 4) + 4 (lane / 32) + r % 4),
// in its two stages
template <int G, int EPI, int WM, int WK>
using TileEpilogueOperands = EpilogueOperands<G, EPI, kOwnedRows<WK>>;

template <int G, int EPI, int WM, int WK>
__device__ __forceinline__ void tile_epilogue_fetch(const CellLevelArgs& a, const int m0, const int j0, const int* sidx,
                                                    TileEpilogueOperands<G, EPI, WM, WK>& eo) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave % WM, wk = wave / WM;
  epilogue_fetch<G, EPI, kOwnedRows<WK>>(
      a, j0 + (lane & 31),
      [&](int v) {
        const int r = tile_acc_row<WK>(wk, v);
        return m0 + wm * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
      },
      eo, sidx, 32 * WM, m0);
}
template <int G, int EPI, int WM, int WK>
__device__ __forceinline__ void tile_epilogue_apply(const CellLevelArgs& a, const int j0,
                                                    const float (&own)[G][kOwnedRows<WK>],
                                                    const TileEpilogueOperands<G, EPI, WM, WK>& eo) {
  epilogue_apply<G, EPI, kOwnedRows<WK>>(
      a, j0 + (int)(threadIdx.x & 31), [&](int g, int v) { return own[g][v]; }, eo);
}

}  // namespace
}  // namespace acrobat
