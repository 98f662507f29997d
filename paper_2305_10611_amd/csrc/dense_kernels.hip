// Wide products with input rows on the fp16 matrix cores at fp32 precision (gfx950): leaf levels and hoisted input
// transforms (of a bidirectional recurrence for both directions in one launch), with the weights kept in registers.
//
// Two launches.  pack_rows_kernel finds every input row's scale, splits the row (split_fp16.h) and stores blocks of 16
// rows as matrix operands, in the order in which the lanes of a matrix instruction want them.  cell_dense_kernel then
// deals the blocks out to groups of workgroups that hold all weights between them - 16 CH hidden units, all gates, each -
// and streams them past: contiguous loads of 1 KB, no LDS on the operands' way, no barrier but the one behind a block's
// partial sums.
// Bound: the matrix cores, as far as the power limit lets them run (a large fp16 product reaches 1.3 PFLOP/s here).  The
// tiled kernel (cell_split_kernels.hip) moves 52 KB through the LDS for every 288 cycles of matrix instructions and is
// bound by that.
// Wavefront w takes K slice w % KS (32-k steps ks, ks + KS, ...) of unit block w / KS; the KS partial sums meet in LDS
// (two buffers), where each thread finishes one element.
#include "dense_kernels.h"

#include "cell_epilogue.h"
#include "packed_rows.h"
#include "split_fp16.h"

#include <algorithm>
#include <atomic>
#include <type_traits>

namespace acrobat {
namespace {

// One workgroup per block of 16 rows: wavefront w takes the 32-k steps w, w + 4, ...
template <int NS>
__global__ __launch_bounds__(256) void pack_rows_kernel(const PackRowsArgs p) {
  __shared__ __attribute__((aligned(16))) float tiles[4][kTurnFloats];
  __shared__ float s_max[4][16];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int T = p.K >> 5, block = blockIdx.x;
  const float* row[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {  // rows past the last repeat it; nothing they give is used
    int i = 16 * block + (lane >> 3) + 8 * h;
    i = i < p.n ? i : p.n - 1;
    row[h] = p.src + (size_t)(p.idx ? p.idx[i] : i) * (size_t)p.K + 4 * (lane & 7);
  }
  floatx4 raw[NS][2];
#pragma unroll
  for (int t = 0; t < NS; ++t) {
    const int step = w + 4 * t;
#pragma unroll
    for (int h = 0; h < 2; ++h)
      raw[t][h] = step < T ? *reinterpret_cast<const floatx4*>(row[h] + 32 * step) : floatx4{0.0f, 0.0f, 0.0f, 0.0f};
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    float m = 0.0f;
#pragma unroll
    for (int t = 0; t < NS; ++t) m = largest(raw[t][h], m);
    m = largest_of_line(m);
    if ((lane & 7) == 0) s_max[w][(lane >> 3) + 8 * h] = m;
  }
  __syncthreads();
  float sc[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int r = (lane >> 3) + 8 * h;
    sc[h] = scale_for(fmaxf(fmaxf(s_max[0][r], s_max[1][r]), fmaxf(s_max[2][r], s_max[3][r])));
    if (w == 0 && (lane & 7) == 0) p.inverse[16 * block + r] = inverse_power(sc[h]);
  }
  if (w == 0) {
    float m = inverse_power(fminf(sc[0], sc[1]));
#pragma unroll
    for (int d = 8; d < 64; d *= 2) m = fmaxf(m, __shfl_xor(m, d));
    if (lane == 0) p.largest[block] = m;
  }
  unsigned char* const dst = static_cast<unsigned char*>(p.operand) + (size_t)block * (64u * p.K) + 16 * lane;
#pragma unroll
  for (int t = 0; t < NS; ++t) {
    const int step = w + 4 * t;
    if (step >= T) break;
    half8 hi, lo;
    turn_write(tiles[w], lane, raw[t], sc[0], sc[1]);
    turn_read(tiles[w], lane, hi, lo);
    *reinterpret_cast<half8*>(dst + (size_t)2048 * step) = hi;
    *reinterpret_cast<half8*>(dst + (size_t)2048 * step + 1024) = lo;
  }
}

// G column tiles of 16 (the gates, or for a single gate G blocks of units), NS steps a wavefront, CH blocks of units a workgroup
template <int G, int EPI, int NS, int CH>
struct DenseShape {
  static constexpr int NW = 8, KS = NW / CH, RB = 2 / CH;  // RB blocks of rows between two barriers: 512 elements
  static constexpr int ZQ = 1024;                          // floats of one wavefront's partial sums of a row block
  static constexpr size_t kLdsBytes = (size_t)2 * RB * NW * ZQ * sizeof(float);
};

template <int G, int EPI, int NS, int CH>
__global__ __launch_bounds__(512, 2) void cell_dense_kernel(const DenseArgs s) {
  using S = DenseShape<G, EPI, NS, CH>;
  constexpr int NW = S::NW, KS = S::KS, RB = S::RB, ZQ = S::ZQ;
  constexpr bool kTiles = EPI == EPI_STORE_Z1;
  static_assert(G <= 4, "the tiles of an element are one vector");
  extern __shared__ __attribute__((aligned(16))) float zbuf[];  // [2][RB][NW][ZQ]
  __shared__ __attribute__((aligned(16))) float s_bias[CH][16][4];
  __shared__ __attribute__((aligned(16))) float s_winv[NW][16][4];

  // Workgroup ids that agree modulo 8 share an XCD: the groups follow one another through the XCDs, so that the members of
  // most find their rows in one L2 and no compute unit stays without work for that.
  const int at = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  const int group = at / s.n_cb, cb = at % s.n_cb;
  if (group >= s.n_groups) return;
  const CellLevelArgs& a = s.two && (group & 1) ? s.b : s.a;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ks = w % KS, ch = w / KS;
  const int li = lane & 15, kq = lane >> 4;
  const int H = a.H, K = a.kseg, T = K >> 5;  // 32-k steps, at most KS * NS
  const int blocks = (a.n + 15) >> 4;
  const int share = s.two ? group >> 1 : group, shares = s.two ? s.n_groups >> 1 : s.n_groups;
  const int b0 = (int)((long)blocks * share / shares), b1 = (int)((long)blocks * (share + 1) / shares);
  if (b0 >= b1) return;
  // first weight row of tile g of unit block c of this workgroup
  const auto tile_row = [&](int g, int c) {
    return kTiles ? 16 * ((cb * CH + c) * G + g) : gate_row<EPI>(g) * H + 16 * (cb * CH + c);
  };

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
        if ((lane & 7) == 0) s_winv[w][(lane >> 3) + 8 * h][g] = inverse_power(sc[h]);
      }
      if (ks == 0 && lane < 16) s_bias[ch][li][g] = a.bias ? a.bias[tile_row(g, ch) + li] : 0.0f;
#pragma unroll
      for (int t = 0; t < NS; ++t) {
        turn_write(tile, lane, raw[g][t], sc[0], sc[1]);
        turn_read(tile, lane, whi[g][t], wlo[g][t]);
      }
    }
  }

  // the element this thread finishes: row er of a row block, unit j
  const int half = w >> 2, er = (tid & 255) >> 4, eu = tid & 15;
  const int my_ch = CH == 2 ? half : 0, my_rb = CH == 2 ? 0 : half;
  const int jb = cb * CH + my_ch, j = 16 * jb + eu;
  const __amdgpu_buffer_rsrc_t operand = agent_buffer(s.operand, s.operand_bytes);
  const unsigned block_bytes = 64u * K;
  constexpr unsigned kNowhere = 0xfffff000u;
  const __amdgpu_buffer_rsrc_t places = agent_buffer(s.places.operand, s.places.operand ? s.places.operand_bytes : 0u);
  ACROBAT_GLOBAL int* const out_rows = keep(const_cast<int*>(a.out_rows));
  ACROBAT_GLOBAL int* const place = keep(const_cast<int*>(s.places.place));
  ACROBAT_GLOBAL float* const inverse = keep(s.inverse);
  floatx4 ring[NS][2];
  auto request = [&](unsigned at, int t) {
    const int step = ks + KS * t;
    at = step < T ? at + 2048u * step : kNowhere;
    ring[t][0] = load_buffer_f4(operand, at + 16u * lane);
    ring[t][1] = load_buffer_f4(operand, at + 16u * lane + 1024u);
  };
  auto block_at = [&](int b) { return b < b1 ? (unsigned)b * block_bytes : kNowhere - 2048u * KS * NS; };
  __syncthreads();
#pragma unroll
  for (int t = 0; t < NS; ++t) {
    request(block_at(b0), t);
    hold_order();
  }
  // Rows whose inverse scale is above `limit` (both are positive: compared as integers) are not to be split against some column
  // of this workgroup.  It does not depend on the other rows of a block, so neither do a row's bits.
  // `some_plain`: the share has such rows.
  const __attribute__((address_space(4))) int* const largest_of = (const __attribute__((address_space(4))) int*)s.largest;
  int limit;
  bool some_plain;
  {
    int most = 0;
    for (int b = b0 + lane; b < b1; b += 64) most = max(most, __float_as_int(s.largest[b]));
    float m = 0.0f;
#pragma unroll
    for (int i = lane; i < 16 * NW; i += 64) {
      const floatx4 u = *reinterpret_cast<const floatx4*>(s_winv[i >> 4][i & 15]);
#pragma unroll
      for (int g = 0; g < G; ++g) m = fmaxf(m, u[g]);
    }
#pragma unroll
    for (int d = 1; d < 64; d *= 2) m = fmaxf(m, __shfl_xor(m, d));
    limit = __builtin_amdgcn_readfirstlane(__float_as_int(kLargestUnit / m));
    some_plain = __ballot(most > limit) != 0;
  }
  // This wavefront's partial sums of the rows of a block that are not to be split, on the fp32 matrix cores.  Bound: the weights
  // that every block fetches again (unscaled features of 1e5, BiRNN, H = D = 512, 300 sequences: 292 us a call on fp32 tiles, 279
  // with these, 1 815 with a scalar product per element; LSTM, 13 402 rows 870 against 7 785 with scalar products).
  auto multiply_plain = [&](int b, floatx4 (&sums)[G]) {
    int i = 16 * b + li;
    i = i < a.n ? i : a.n - 1;
    const float* const x = a.src0 + (size_t)(a.idx0 ? a.idx0[i] : i) * (size_t)a.ld0 + 4 * kq;
    floatx4 acc[G];
#pragma unroll
    for (int g = 0; g < G; ++g) acc[g] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
    for (int half = 2 * ks; half < 2 * T; half = half & 1 ? half + 2 * KS - 1 : half + 1) {  // 16 k at a time
      const floatx4 xk = *reinterpret_cast<const floatx4*>(x + 16 * half);
      floatx4 wk[G];
#pragma unroll
      for (int g = 0; g < G; ++g)
        wk[g] = *reinterpret_cast<const floatx4*>(a.W + (size_t)(tile_row(g, ch) + li) * (size_t)a.ldw + 4 * kq + 16 * half);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int g = 0; g < G; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(xk[e], wk[g][e], acc[g], 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const bool plain = __float_as_int(at_byte(inverse, 4u * (unsigned)(16 * b + 4 * kq + v))) > limit;
#pragma unroll
      for (int g = 0; g < G; ++g) sums[g][v] = plain ? acc[g][v] : sums[g][v];
    }
  };
  int parity = 0;
  for (int b = b0; b < b1; b += RB, parity ^= 1) {
    int i = 16 * (b + my_rb) + er;
    const bool live = i < a.n && b + my_rb < b1;
    i = i < a.n ? i : a.n - 1;
    const int out = out_rows ? at_byte(out_rows, 4u * (unsigned)i) : i;
    int to = -1;
    if (EPI == EPI_TREE_LEAF && place) to = at_byte(place, 4u * (unsigned)i);
    const float rinv = at_byte(inverse, 4u * (unsigned)i);
    float* const zc = zbuf + parity * (RB * NW * ZQ);
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      floatx4 acc[G];
#pragma unroll
      for (int g = 0; g < G; ++g) acc[g] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
      const unsigned next = block_at(b + r + 1);
#pragma unroll
      for (int t = 0; t < NS; ++t) {
        const half8 hi = __builtin_bit_cast(half8, ring[t][0]), lo = __builtin_bit_cast(half8, ring[t][1]);
#pragma unroll
        for (int g = 0; g < G; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(lo, whi[g][t], acc[g], 0, 0, 0);
#pragma unroll
        for (int g = 0; g < G; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hi, wlo[g][t], acc[g], 0, 0, 0);
#pragma unroll
        for (int g = 0; g < G; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hi, whi[g][t], acc[g], 0, 0, 0);
        hold_order();
        request(next, t);
        hold_order();
      }
      const floatx4 unit = *reinterpret_cast<const floatx4*>(s_winv[w][li]);
#pragma unroll
      for (int g = 0; g < G; ++g) acc[g] *= unit[g];
      if (__builtin_expect(some_plain && b + r < b1 && largest_of[b + r] > limit, 0)) multiply_plain(b + r, acc);
      float* const z = zc + (r * NW + w) * ZQ;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        floatx4 part = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int g = 0; g < G; ++g) part[g] = acc[g][v];
        *reinterpret_cast<floatx4*>(z + ((4 * kq + v) * 16 + li) * 4) = part;
      }
    }
    // (a buffer written two rounds ago has been read: its readers have passed the barrier in between)
    __syncthreads();
    const float* const zr = zc + (my_rb * NW + my_ch * KS) * ZQ + (er * 16 + eu) * 4;
    floatx4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int q = 0; q < KS; ++q) {
      const floatx4 part = *reinterpret_cast<const floatx4*>(zr + q * ZQ);
#pragma unroll
      for (int g = 0; g < G; ++g) sum[g] += part[g];
    }
    if (!live) continue;
    // scales out again (of what was split); what is not finite is computed in fp32, term by term
    const float scale = __float_as_int(rinv) > limit ? 1.0f : rinv;
    float zs[G];
    bool bad = false;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      zs[g] = sum[g] * scale;
      bad |= !__builtin_isfinite(zs[g]);
    }
    if (__builtin_expect(bad, 0)) {
      const float* const x = a.src0 + (size_t)(a.idx0 ? a.idx0[i] : i) * (size_t)a.ld0;
#pragma unroll 1
      for (int g = 0; g < G; ++g) {
        const float* const wr = a.W + (size_t)(tile_row(g, my_ch) + eu) * (size_t)a.ldw;
        float z = 0.0f;
#pragma unroll 1
        for (int k = 0; k < K; k += 4) {
          const floatx4 xk = *reinterpret_cast<const floatx4*>(x + k), wk = *reinterpret_cast<const floatx4*>(wr + k);
#pragma unroll
          for (int c = 0; c < 4; ++c) z = __builtin_fmaf(xk[c], wk[c], z);
        }
#pragma unroll
        for (int e = 0; e < G; ++e) zs[e] = e == g ? z : zs[e];
      }
    }
    const floatx4 bias = *reinterpret_cast<const floatx4*>(s_bias[my_ch][eu]);
    if constexpr (EPI == EPI_STORE_Z) {
#pragma unroll
      for (int g = 0; g < G; ++g) a.zout[(size_t)out * (size_t)(G * H) + g * H + j] = zs[g] + bias[g];
    } else if constexpr (kTiles) {
#pragma unroll
      for (int g = 0; g < G; ++g) a.zout[(size_t)out * (size_t)H + tile_row(g, my_ch) + eu] = zs[g] + bias[g];
    } else {
      const float c = fast_sigmoid(zs[0] + bias[0]) * fast_tanh(zs[2] + bias[2]);
      const float h = fast_sigmoid(zs[1] + bias[1]) * fast_tanh(c);
      a.c[(size_t)out * H + j] = c;
      a.h[(size_t)out * H + j] = h;
      if (place) store_tree_place(places, s.places.cells, H, to, jb, eu, lane, h, c);
    }
  }
}

template <int G, int EPI, int NS, int CH>
struct Dense {
  static constexpr size_t kLdsBytes = DenseShape<G, EPI, NS, CH>::kLdsBytes;
  static constexpr int kUnits = 16 * CH * (EPI == EPI_STORE_Z1 ? G : 1);
  static hipError_t launch(DenseArgs s, int n_cu, hipStream_t stream, const LaunchEvents& ev) {
    static std::atomic<uint64_t> configured{0};  // (see tree_kernels.hip)
    int dev = 0;
    if (const hipError_t e = hipGetDevice(&dev); e != hipSuccess) return e;
    const uint64_t bit = 1ull << (dev & 63);
    if (dev >= 64 || !(configured.load(std::memory_order_acquire) & bit)) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&cell_dense_kernel<G, EPI, NS, CH>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBytes);
      if (e != hipSuccess) return e;
      if (dev < 64) configured.fetch_or(bit, std::memory_order_release);
    }
    // one workgroup per compute unit in groups of H / kUnits (nobody waits for anybody)
    s.n_cb = s.a.H / kUnits;
    s.n_groups = n_cu / s.n_cb;
    const int blocks = (s.a.n + 15) / 16 * (s.two ? 2 : 1);
    if (s.n_groups > blocks) s.n_groups = blocks;
    if (s.n_groups < 1) s.n_groups = 1;
    if (s.two) s.n_groups = s.n_groups < 2 ? 2 : s.n_groups & ~1;
    const unsigned grid = 8u * (unsigned)((s.n_groups * s.n_cb + 7) / 8);
    launch_with_events((cell_dense_kernel<G, EPI, NS, CH>), dim3(grid), dim3(512), kLdsBytes, stream, ev.start, ev.stop, s);
    return hipGetLastError();
  }
};

template <int G, int EPI>
hipError_t launch_gates(const DenseArgs& s, int n_cu, hipStream_t stream, const LaunchEvents& ev) {
  const int K = s.a.kseg;
  if (K <= 128) return Dense<G, EPI, 1, 2>::launch(s, n_cu, stream, ev);
  if (K <= 256) return Dense<G, EPI, 2, 2>::launch(s, n_cu, stream, ev);
  if (K <= 384) return Dense<G, EPI, 3, 2>::launch(s, n_cu, stream, ev);
  if (K <= 512) return Dense<G, EPI, 4, 2>::launch(s, n_cu, stream, ev);
  if (K <= 768) return Dense<G, EPI, 3, 1>::launch(s, n_cu, stream, ev);
  return Dense<G, EPI, 4, 1>::launch(s, n_cu, stream, ev);
}

}  // namespace

bool dense_level_wins(CellEpilogue epi, int32_t n, int32_t H, int32_t K, const SplitKWorkspace& ws) {
  if ((epi != EPI_TREE_LEAF && epi != EPI_STORE_Z && epi != EPI_STORE_Z1) || n <= 0 || K <= 0 || K > kDenseMaxK || ws.force_bm ||
      (double)((n + 15) / 16) * 64 * K > kDenseMaxBytes)
    return false;
  // Two launches, and all weights fetched by every group, have to be earned.  Leaf levels, whole calls, stationary kernel
  // against this one: 1 000 leaves, H = D = 512 (1.6 GFLOP) 74.8 and 72.6 us, 2 500 102.5 and 92.6, 250 (0.4) 49.7 and 51.7;
  // 2 500, H = D = 256 (1.0) 60.1 and 62.3.  LSTM input products, fp32 tiles against this one: 250 rows, H = 512, D = 1024
  // (1.0) 50.2 and 48.4, D = 512 (0.5) 37.2 and 42.7; 750, H = D = 320 (0.6) 40.4 and 41.8.  Small models have fewer columns for
  // every packed row: leaves, split tiles against this one, 22 000, H = D = 192 211 and 217; H = 256, D = 544 295 and 294;
  // input products, 10 000 rows, H = 192, D = 160 87 and 90, H = 256 101 and 98.
  // Both directions of a bidirectional recurrence in one launch, fp32 tiles against this one: 3 000 rows, H = D = 256 (0.8)
  // 56.8 and 58.3, H = D = 320 (1.2) 65.7 and 66.5, D = 512, H = 256 (1.6) 61.8 and 61.0; 6 000, H = D = 256 (1.6) 76.8 and
  // 73.3, H = D = 512 (6.3) 137 and 111; 1 200 rows, H = D = 512 (1.3), the product alone, 21 and 23; short rows: 6 000, D = 128,
  // H = 512 (1.6) 102 and 104; H = 128 loses throughout (18 000 rows 126 and 136).
  if (H < 256) return false;
  if (epi == EPI_STORE_Z1) return H % 64 == 0 && K >= 256 && 4.0 * n * H * K >= 1.5e9;
  return 2.0 * (epi == EPI_TREE_LEAF ? 3 : 4) * n * H * K >= 1.0e9;
}

namespace {

hipError_t launch_rows(CellEpilogue epi, DenseArgs s, void* scratch, int n_cu, hipStream_t stream, const LaunchEvents& ev) {
  PackRowsArgs p{s.a.n, s.a.kseg, s.a.src0, s.a.idx0, scratch, nullptr, nullptr};
  const unsigned blocks = (unsigned)((p.n + 15) / 16);
  s.operand = scratch;
  s.operand_bytes = 64u * (unsigned)p.K * blocks;
  p.inverse = s.inverse = reinterpret_cast<float*>(static_cast<unsigned char*>(scratch) + (size_t)s.operand_bytes);
  s.largest = p.largest = p.inverse + (size_t)16 * blocks;
  if (p.K <= 128) launch_with_events((pack_rows_kernel<1>), dim3(blocks), dim3(256), 0, stream, ev.start, hipEvent_t(nullptr), p);
  else if (p.K <= 256) launch_with_events((pack_rows_kernel<2>), dim3(blocks), dim3(256), 0, stream, ev.start, hipEvent_t(nullptr), p);
  else if (p.K <= 512) launch_with_events((pack_rows_kernel<4>), dim3(blocks), dim3(256), 0, stream, ev.start, hipEvent_t(nullptr), p);
  else launch_with_events((pack_rows_kernel<8>), dim3(blocks), dim3(256), 0, stream, ev.start, hipEvent_t(nullptr), p);
  if (const hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  LaunchEvents second;
  second.stop = ev.stop;
  if (epi == EPI_STORE_Z1) {
    const int K = s.a.kseg;
    if (K <= 256) return Dense<4, EPI_STORE_Z1, 1, 1>::launch(s, n_cu, stream, second);
    if (K <= 512) return Dense<4, EPI_STORE_Z1, 2, 1>::launch(s, n_cu, stream, second);
    return Dense<4, EPI_STORE_Z1, 4, 1>::launch(s, n_cu, stream, second);
  }
  return epi == EPI_TREE_LEAF ? launch_gates<3, EPI_TREE_LEAF>(s, n_cu, stream, second)
                              : launch_gates<4, EPI_STORE_Z>(s, n_cu, stream, second);
}

}  // namespace

hipError_t launch_dense_level(CellEpilogue epi, const DenseArgs& s, void* scratch, size_t scratch_bytes, int n_cu,
                              hipStream_t stream, const LaunchEvents& ev) {
  const size_t rows = scratch_bytes / dense_scratch_bytes(16, s.a.kseg) * 16;
  if (rows >= (size_t)s.a.n) return launch_rows(epi, s, scratch, n_cu, stream, ev);
  if (epi != EPI_TREE_LEAF || rows == 0 || !s.a.idx0 || !s.a.out_rows) return hipErrorInvalidValue;
  const int pieces = (int)((s.a.n + rows - 1) / rows), piece = (s.a.n + 16 * pieces - 1) / (16 * pieces) * 16;  // alike, whole blocks
  for (int at = 0; at < s.a.n; at += piece) {
    DenseArgs p = s;
    p.a.n = std::min(piece, s.a.n - at);
    p.a.idx0 += at;
    p.a.out_rows += at;
    if (p.places.place) p.places.place += at;
    const LaunchEvents some{at == 0 ? ev.start : nullptr, at + piece >= s.a.n ? ev.stop : nullptr};
    if (const hipError_t e = launch_rows(epi, p, scratch, n_cu, stream, some); e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace acrobat
