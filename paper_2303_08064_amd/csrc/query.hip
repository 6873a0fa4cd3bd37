// Fused guiding query: MLP forward on MFMA (weights LDS-resident), NASG
// decode, inverse-CDF lobe choice, direct sampling (App. C) and the mixture
// pdf at the sampled direction (Sec. 3.1), in 16-vertex blocks.
//
// Lane (g, c) of a wave owns vertex c of a 16-vertex block and lobes
// g*K/4 .. g*K/4 + K/4 - 1 of that vertex, so reductions over lobes are a
// within-lane loop plus two cross-lane steps (xor 16, xor 32). A wave takes
// one block per pass, four (one sample per lane) or two
// (the paper's network), with the multi-block passes' inputs staged in LDS
// one pass ahead.
#include <type_traits>

#include "epilogue.hpp"
#include "kernels.hpp"
#include "mlp.hpp"

namespace nasg {

// 16-vertex blocks per wave pass (NB of the kernels below):
// * 4, the hidden-64 networks' queries of large batches: one sample per lane
//   (the four blocks' lobes take 144 registers at K = 16, so two waves per
//   SIMD): BF16 in two workgroups of four waves per CU, FP32 (weights of up to
//   61 KiB, K = 4, to 90, K = 16 with selection) in one of eight;
// * 1, their queries of small batches (query_is_small) and raw forwards;
// * 2, the hidden-128 network whose 132 KiB of forward weights leave room for
//   one workgroup per CU: eight waves, every weight fragment read feeds both
//   blocks.
// dynamic LDS of a query launch: the weights, plus the multi-block kernels'
// two input staging buffers per wave
constexpr size_t query_dynamic_lds(int weight_bytes, int nb, int nw) {
  return (size_t)weight_bytes + (nb > 1 ? (size_t)nw * 2 * (kInFeatures + 4) * kTileV * nb * sizeof(float) : 0);
}
constexpr int query_waves_per_eu(int NB, int MODE, int PREC, int K) {
  return NB == 1 ? (MODE == 1 ? 1 : (PREC == 1 && K < 16 ? 3 : 2)) : 2;
}

// MODE 1: store a 16-vertex block's raw outputs in canonical row order.
template <int K, int S, int MTO>
__device__ __forceinline__ void store_raw(const QueryArgs& a, const float (&out)[MTO][4], int64_t v, int g) {
  constexpr int KQ = K / 4;
  if (v >= a.B) return;
  // accumulator t of lane group g is parameter t / KQ of lobe g*KQ + t % KQ
#pragma unroll
  for (int t = 0; t < 2 * K; ++t) {
    int p = t / KQ, k = g * KQ + t % KQ;
    a.raw_out[(int64_t)(p * K + k) * a.ld + v] = out[t >> 2][t & 3];
  }
  if (S == 1 && g == 0) a.raw_out[(int64_t)(8 * K) * a.ld + v] = out[MTO - 1][0];
}

// Inputs of one 64-vertex pass staged in LDS: the 9 feature rows and the 4
// uniform rows, 64 floats each (lane i of a row = vertex 64 tile + i).
constexpr int kPassRows = kInFeatures + 4;
constexpr int kPassStage = kPassRows * 64;   // floats per wave and buffer

// Direct-to-LDS copies of a pass's inputs (13 wave instructions, no
// registers). Lanes past the batch read vertex B - 1 instead (in bounds; it is
// computed and its results are not stored), so that every wave issues the same
// number of copies and s_waitcnt can count them.
__device__ __forceinline__ void stage_pass(const QueryArgs& a, int64_t tile, float* buf, int lane) {
  int64_t v = tile * (4 * kTileV) + lane;
  v = v < a.B ? v : a.B - 1;
#pragma unroll
  for (int k = 0; k < kInFeatures; ++k)
    __builtin_amdgcn_global_load_lds(a.feat + k * a.ld + v, (__attribute__((address_space(3))) void*)(buf + k * 64), 4,
                                     0, 0);
#pragma unroll
  for (int k = 0; k < 4; ++k)
    __builtin_amdgcn_global_load_lds(a.xi + k * a.ld + v,
                                     (__attribute__((address_space(3))) void*)(buf + (kInFeatures + k) * 64), 4, 0, 0);
}

// The same for a 32-vertex pass (two 16-vertex blocks): each copy moves two
// rows, lanes 0-31 the first and 32-63 the second (lanes past the last row
// copy nothing); the uniforms only for a query (XI). ceil(rows / 2) copies.
template <bool XI>
__device__ __forceinline__ void stage_pass32(const QueryArgs& a, int64_t tile, float* buf, int lane) {
  constexpr int rows = kInFeatures + (XI ? 4 : 0);
  int64_t v = tile * (2 * kTileV) + (lane & 31);
  v = v < a.B ? v : a.B - 1;
#pragma unroll
  for (int j = 0; j < (rows + 1) / 2; ++j) {
    const int r = 2 * j + (lane >> 5);
    if (r < rows) {
      const float* src = r < kInFeatures ? a.feat + r * a.ld + v : a.xi + (r - kInFeatures) * a.ld + v;
      __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void*)(buf + 2 * j * 32), 4, 0, 0);
    }
  }
}

// MODE 0: query, 1: raw forward only, 2: query that also stores the decoded
// records (a kernel of its own: the store's addresses and the raw outputs
// that it needs raise the K = 16 kernel from 224 to 256 registers); S = 1:
// the network has the selection output (row 8K, read by lane group 0 from
// the extra output tile); E = 1: the encoded input; NB: 16-vertex blocks per
// wave per pass; NW: waves per workgroup.
// Bound by VALU issue (the K = 16 BF16 pass of 64 vertices issues 4460 slots,
// 4864 before log K, the log-sum-exp and the base-e scalings went, see
// decode_lobe_query and query_sum). Measured against one block a pass, the
// log-sum-exp and loads behind branches: 2^20 K = 16 BF16 queries 145 -> 131 us,
// K = 8 103 -> 89 us, 120000 FP32 K = 8 queries with records 54.1 -> 48.2 us,
// 600000 of the hidden-128 network 111 -> 100 us (one sample per two lane
// groups, was per group), 777 K = 4 BF16 queries 9.3 -> 4.0 us (the kernel).
template <int H, int K, int PREC, int MODE, int S, int E, int NB, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(query_waves_per_eu(NB, MODE, PREC, K))))
void query_kernel(QueryArgs a) {
  constexpr int NHMAX = 4;
  typedef Mlp<H, K, PREC, E> M;
  typedef Forward<H, K, PREC, NHMAX, S, E> F;
  typedef typename F::W W;
  extern __shared__ __align__(16) unsigned char smem[];
  W* lds = reinterpret_cast<W*>(smem);
  // the forward weights by direct-to-LDS loads: every wave's copies are in
  // flight at once (a register round trip per 16 bytes waited on each load)
  lds_dma(lds, a.wpack, a.lds_bytes);
  constexpr int KQ = K / 4;
  constexpr bool REC = MODE == 2;
  // block-major MFMAs: 1-3% faster than row tile by row tile, but for the
  // four-block K = 16 kernel (1% slower: 254 registers)
  constexpr bool BM = !(NB == 4 && K == 16);

  const int lane = lane_id();
  const int g = lane >> 4, c = lane & 15;
  const int wave = threadIdx.x >> 6;
  // inputs of one block of a one-block pass, without branches (a branch waits
  // for its loads); lanes past the batch read, as in the staged passes, its
  // last vertex, and their results are not stored
  struct BlockIn {
    typename M::Raw x;
    float xi[4];
  };
  auto load_block = [&](int64_t block) {
    BlockIn in;
    int64_t v = block * kTileV + c;
    v = v < a.B ? v : a.B - 1;
    in.x = M::load_raw(a.feat, a.ld, v, g);
#pragma unroll
    for (int r = 0; r < 4; ++r) in.xi[r] = MODE != 1 ? a.xi[r * a.ld + v] : 0.0f;
    return in;
  };
  // one-block passes: four waves of a workgroup (one per SIMD) take
  // neighbouring blocks (64 bytes of every row each); a workgroup's second
  // four come after everyone's first, so that the end of a batch runs one
  // wave per SIMD. The first block's inputs are requested beside the weights.
  int64_t block = (int64_t)(wave >> 2) * 4 * gridDim.x + (int64_t)blockIdx.x * 4 + (wave & 3);
  BlockIn first;
  if constexpr (NB == 1) first = load_block(block);
  lds_dma_wait();
  __syncthreads();
  const W* wts = lds;
  if constexpr (NB == 4) {
    // each wave's two staging buffers follow the weights: the next pass's
    // inputs are copied while this pass runs, so no block waits for memory
    float* stage = reinterpret_cast<float*>(smem + a.lds_bytes) + wave * 2 * kPassStage;
    const int64_t n_tiles = (a.B + 4 * kTileV - 1) / (4 * kTileV);
    const int64_t stride = (int64_t)gridDim.x * NW;
    int64_t tile = (int64_t)blockIdx.x * NW + wave;
    if (tile < n_tiles) stage_pass(a, tile, stage, lane);
    for (int p = 0; tile < n_tiles; tile += stride, p ^= 1) {
      float* cur = stage + p * kPassStage;
      if (tile + stride < n_tiles) {
        stage_pass(a, tile + stride, stage + (p ^ 1) * kPassStage, lane);
        // the current pass's 13 copies and everything before them are done;
        // the 13 just issued may still be in flight
        __builtin_amdgcn_s_waitcnt(0x0F70 | 13);
      } else {
        lds_dma_wait();
      }
      // the forward runs block by block, each block's decoded lobes kept
      // until the four blocks' vertices have been sampled, one per lane. The
      // next block's forward stays out of a block's decode where the
      // scheduler's mix of the two spills (FP32, and K = 16 with the
      // selection tile or the record store); elsewhere the mix is 1% faster
      constexpr bool SPLIT = PREC == 0 || (K == 16 && (REC || S == 1));
      query_epilogue<KQ, S, 4, REC, SPLIT, F::MTO>(
          a, tile * (4 * kTileV), lane,
          [&](int b, float (&out)[F::MTO][4]) {
            const typename M::Input x = M::input(M::load_raw(cur, 64, b * kTileV + c, g), true, g);
            F::template run_query<BM>(wts, a.nh, x, out, lane);
          },
          [&](int r, int i) { return cur[(kInFeatures + r) * 64 + i]; });
    }
    return;
  }
  constexpr int TV = kTileV * NB;   // vertices per wave pass
  const int64_t n_tiles = (a.B + TV - 1) / TV;
  const int64_t stride = (int64_t)gridDim.x * NW;
  if constexpr (NB == 1) {
    for (BlockIn in = first; block < n_tiles; in = load_block(block)) {
      const typename M::Input x = M::input(in.x, true, g);
      if constexpr (MODE == 1) {
        float out[F::MTO][4];
        F::template run_query<BM>(wts, a.nh, x, out, lane);
        store_raw<K, S>(a, out, block * kTileV + c, g);
      } else {
        query_epilogue<KQ, S, 1, REC, false, F::MTO>(
            a, block * kTileV, lane, [&](int, float (&out)[F::MTO][4]) { F::template run_query<BM>(wts, a.nh, x, out, lane); },
            [&](int r, int) { return in.xi[r]; });
      }
      block += stride;
    }
  } else if constexpr (NB == 2) {
    // two 16-vertex blocks per pass, their inputs staged in LDS one pass
    // ahead (as for four): the rows of a pass are [row][32]
    constexpr int ROWS = kInFeatures + (MODE != 1 ? 4 : 0);
    constexpr int COPIES = (ROWS + 1) / 2;
    float* stage = reinterpret_cast<float*>(smem + a.lds_bytes) + wave * 2 * (kPassRows * 32);
    int64_t tile = (int64_t)blockIdx.x * NW + wave;
    if (tile < n_tiles) stage_pass32<MODE != 1>(a, tile, stage, lane);
    for (int p = 0; tile < n_tiles; tile += stride, p ^= 1) {
      const float* cur = stage + p * (kPassRows * 32);
      if (tile + stride < n_tiles) {
        stage_pass32<MODE != 1>(a, tile + stride, stage + (p ^ 1) * (kPassRows * 32), lane);
        __builtin_amdgcn_s_waitcnt(0x0F70 | COPIES);
      } else {
        lds_dma_wait();
      }
      typename M::Input x[NB];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) x[nb] = M::input(M::load_raw(cur, 32, nb * kTileV + c, g), true, g);
      float out[NB][F::MTO][4];
      F::template run_query_nb<NB, MODE != 1>(wts, a.nh, x, out, lane);
      if constexpr (MODE == 1) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) store_raw<K, S>(a, out[nb], tile * TV + nb * kTileV + c, g);
      } else {
        query_epilogue<KQ, S, NB, REC, false, F::MTO>(
            a, tile * TV, lane,
            [&](int b, float (&o)[F::MTO][4]) {
#pragma unroll
              for (int mt = 0; mt < F::MTO; ++mt)
#pragma unroll
                for (int i = 0; i < 4; ++i) o[mt][i] = out[b][mt][i];
            },
            [&](int r, int i) { return cur[(kInFeatures + r) * 32 + i]; });
      }
    }
  }
}

// The kernel of one variant and the workgroups per CU that it reaches.
struct QueryKernel {
  void (*kern)(QueryArgs);
  hipError_t (*set_lds)(size_t);
  int nb, nw;
  size_t max_weights;   // bytes, of the network shape's deepest variant (4 hidden layers)
};

template <int H, int K, int PREC, int MODE, int S, int E, int NB, int NW>
static QueryKernel query_variant() {
  const NetDims dmax{H, 4, K, S, E};
  const size_t w = PREC == 1 ? (size_t)Bf16Layout{dmax}.fwd_elems() * 2 : (size_t)F32Layout{dmax}.total_elems() * 4;
  return {query_kernel<H, K, PREC, MODE, S, E, NB, NW>, set_max_lds_once<query_kernel<H, K, PREC, MODE, S, E, NB, NW>>,
          NB, NW, w};
}

template <int H, int K, int PREC, int MODE, int S>
static QueryKernel net64_variant(bool small) {
  constexpr int NW4 = PREC == 0 ? 8 : 4;
  // one workgroup per CU (K = 16 in FP32): eight waves of one-block passes
  // too, for two per SIMD
  constexpr int NW1 = PREC == 0 && K == 16 && MODE != 1 ? 8 : 4;
  if constexpr (MODE == 1) return query_variant<H, K, PREC, 1, S, 0, 1, NW1>();
  else return small ? query_variant<H, K, PREC, MODE, S, 0, 1, NW1>() : query_variant<H, K, PREC, MODE, S, 0, 4, NW4>();
}
template <int H, int K, int PREC, int S>
static QueryKernel net64_kernel(int mode, bool small) {
  return mode == 0   ? net64_variant<H, K, PREC, 0, S>(small)
         : mode == 1 ? net64_variant<H, K, PREC, 1, S>(small)
                     : net64_variant<H, K, PREC, 2, S>(small);
}

// The resident query kernel of a network; nb = 0 when it has none.
static QueryKernel find_query_kernel(const NetDims& d, int prec, int mode, bool small) {
#define NASG_CASE(h, k, p)                                  \
  if (d.H == h && d.K == k && prec == p && d.E == 0)        \
    return d.S ? net64_kernel<h, k, p, 1>(mode, small) : net64_kernel<h, k, p, 0>(mode, small);
  NASG_FOR_EACH_NET(NASG_CASE)
#undef NASG_CASE
#define NASG_CASE(h, k, p, s, e)                                             \
  if (d.H == h && d.K == k && prec == p && d.S == s && d.E == e)             \
    return mode == 0   ? query_variant<h, k, p, 0, s, e, 2, 8>()             \
           : mode == 1 ? query_variant<h, k, p, 1, s, e, 2, 8>()             \
                       : query_variant<h, k, p, 2, s, e, 2, 8>();
  NASG_FOR_EACH_RESIDENT_QUERY(NASG_CASE)
#undef NASG_CASE
  return {nullptr, nullptr, 0, 0, 0};
}

// One-block or four-block passes, by what the batch's rounds cost. With eight
// waves per CU (two per SIMD) a round of one-block passes takes 128 vertices a
// CU, one of four-block passes 512; a batch's last round counts as half where
// one wave per SIMD is enough for it. In thousandths of a four-block round:
// * BF16, one-block passes: `slope` a half round and an offset, as their rounds
//   overlap (K = 4 and 8 hold three waves per SIMD);
// * BF16, four-block passes: 1000 a round and for a last half `first`, less
//   `drop` for every round before it, but `least` (waves that are out of step
//   by then fill its idle SIMDs);
// * with the record store both cost more; past 220 MB of records, near the size
//   of the last-level cache (256 MB), the four-block passes are the safer ones
//   (K = 16 with selection, 393216 vertices: 78.6 / 72.8 us, without 71.2 / 75.6);
// * FP32, whose chains of 32-cycle MFMAs wait for themselves: 270 a one-block
//   round, 150 its half, a last four-block half as long as a full one.
// Measured (us, one-block / four-block, 256 CUs): K = 16 BF16 49152 vertices
// 9.3 / 14.7, 65536 10.9 / 14.7, 114688 17.4 / 18.6, 131072 18.9 / 18.8, 180224
// 25.0 / 27.1, 196608 27.7 / 27.3, 229376 31.2 / 34.9, 327680 43.8 / 40.6,
// 360448 48.4 / 51.3; with records 65536 14.9 / 21.0, 131072 24.1 / 25.2, 180224
// 31.1 / 36.0, 262144 43.3 / 45.5, 376832 59.4 / 63.4, 442368 91.5 / 88.5. K = 8
// 114688 11.9 / 13.4, 131072 14.1 / 13.4, 245760 22.8 / 24.1, 262144 25.4 / 24.4,
// 475136 43.1 / 45.9, 589824 52.3 / 49.2; with records 131072 17.4 / 18.1, 393216
// 41.2 / 43.5, 786432 91.3 / 94.5, 983040 139 / 125. K = 4 131072 9.7 / 10.5,
// 196608 13.8 / 12.5, 229376 15.2 / 16.6, 262144 17.5 / 16.6; with records 196608
// 16.9 / 16.4, 229376 18.4 / 20.7. FP32 K = 8 777 8.7 / 41, 98304 35.3 / 43.0,
// 131072 45.1 / 43.4, 200000 71 / 83.
static bool query_is_small(int64_t B, int num_cus, int K, int prec, bool records) {
  const int64_t unit = 64LL * num_cus;                          // a one-block half round
  const int64_t h = (B + unit - 1) / unit;                      // one-block half rounds
  const int64_t q = (B + 4 * unit - 1) / (4 * unit);            // four-block half rounds
  if (prec != 1) return 270 * (h / 2) + 150 * (h % 2) < 1000 * ((q + 1) / 2);
  if (records && B * (9 * 4) * K > 220000000) return false;
  struct Cost { int slope, offset, first, drop, least; };
  const Cost c = K == 4   ? (records ? Cost{150, -320, 400, 0, 400} : Cost{157, -350, 350, 0, 350})
                 : K == 8 ? (records ? Cost{120, 20, 780, 140, 200} : Cost{132, -50, 780, 140, 200})
                          : (records ? Cost{123, 0, 770, 250, 250} : Cost{128, 0, 770, 250, 250});
  int64_t four = 1000 * (q / 2);
  if (q % 2) {
    const int64_t last = c.first - c.drop * (q / 2);
    four += last > c.least ? last : c.least;
  }
  return c.slope * h + c.offset < four;
}

hipError_t launch_query(const QueryArgs& a, const NetDims& d, int prec, int mode, hipStream_t st) {
  const bool small = query_is_small(a.B, a.num_cus, d.K, prec, mode == 2);
  const QueryKernel k = find_query_kernel(d, prec, mode, small);
  if (k.nb == 0) return hipErrorInvalidValue;
  const int TV = kTileV * k.nb;   // vertices per wave pass
  const int64_t n_tiles = (a.B + TV - 1) / TV;
  // one-block passes: a workgroup for every four blocks up to the capacity
  const int64_t want = k.nb == 1 ? (n_tiles + 3) / 4 : (n_tiles + k.nw - 1) / k.nw;
  const int per_cu = a.per_cu[small];
  const int64_t cap = (int64_t)(per_cu < 1 ? 1 : per_cu) * a.num_cus;
  const int grid = (int)(want < cap ? (want < 1 ? 1 : want) : cap);
  hipLaunchKernelGGL(k.kern, dim3(grid), dim3(64 * k.nw), query_dynamic_lds(a.lds_bytes, k.nb, k.nw), st, a);
  return hipGetLastError();
}

// The LDS limit is raised once to the footprint of the network shape's
// deepest variant (4 hidden layers); the occupancy is that of the caller's
// footprint.
hipError_t query_workgroups_per_cu(const NetDims& d, int prec, int mode, bool small, int lds_bytes, int* per_cu) {
  const QueryKernel k = find_query_kernel(d, prec, mode, small);
  if (k.nb == 0 || (size_t)lds_bytes > k.max_weights) return hipErrorInvalidValue;
  hipError_t e = k.set_lds(query_dynamic_lds((int)k.max_weights, k.nb, k.nw));
  if (e != hipSuccess) return e;
  int n = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, (const void*)k.kern, 64 * k.nw,
                                                   query_dynamic_lds(lds_bytes, k.nb, k.nw));
  *per_cu = n < 1 ? 1 : n;
  return e;
}

bool query_is_resident(const NetDims& d, int prec) { return find_query_kernel(d, prec, 0, false).nb != 0; }

}  // namespace nasg
