// MLP backward pieces shared by the training kernels: dgrad in registers,
// staging of a layer's deltas and inputs for the weight gradient, the
// weight-gradient MFMA over a workgroup's staged vertices, and the flush of a
// wave's gradient tiles to its workgroup's partial.
//
// dW_l = sum_v delta_l(v) h_{l-1}(v)^T contracts over vertices, which sit in
// different lanes of the accumulator layout, so the waves of a workgroup
// stage delta_l and h_{l-1} of its vertices in LDS, and each wave accumulates
// its own tiles of dW_l.
#pragma once

#include <type_traits>

#include "common.hpp"
#include "mlp.hpp"

namespace nasg {

constexpr int kWGV = 64;   // vertices per workgroup tile

// delta_prev = W_l^T delta (contraction over the RT*16 rows of layer l),
// rows of the result are the previous layer's neurons in accumulator layout.
template <int H, int K, int PREC, int RT>
__device__ __forceinline__ void dgrad(const void* wl, const float (&dl)[RT][4],
                                      float (&dp)[H / 16][4], int lane) {
  constexpr int MTP = H / 16;
  if constexpr (PREC == 1) {
    constexpr int KB = RT / 2;   // 32-wide blocks over the rows of layer l
    const bf16x8* frag = reinterpret_cast<const bf16x8*>(wl);
    bf16x8 b[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int j = 0; j < 8; ++j) b[kb][j] = (__bf16)dl[2 * kb + (j >> 2)][j & 3];
    // an odd last row tile (the selection tile) contracts with 16x16x16
    // fragments stored after the 32-wide ones: lane (g, c) holds its rows
    // 4g .. 4g+3, which are this lane's accumulators dl[RT-1][0..3]. Its
    // product has an accumulator of its own, added with VALU: chaining a
    // 16x16x16 MFMA onto a 16x16x32 accumulator gave non-reproducible
    // results with this toolchain.
    const bf16x4* frag_s = reinterpret_cast<const bf16x4*>(frag + MTP * KB * 64);
    bf16x4 bs;
    if constexpr (RT % 2 == 1) {
#pragma unroll
      for (int j = 0; j < 4; ++j) bs[j] = (__bf16)dl[RT - 1][j];
    }
    // block-major with prefetched fragments (mfma_rows): the chains of the
    // MTP row tiles interleave instead of waiting on each other
    f32x4 acc[1][MTP];
    mfma_rows<MTP, KB, 1>(frag, [&](int, int kb) { return b[kb]; }, acc, lane);
#pragma unroll
    for (int mt = 0; mt < MTP; ++mt) {
      if constexpr (RT % 2 == 1) {
        const f32x4 sel = mfma_bf16_16(frag_s[mt * 64 + lane], bs, zero4());
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[0][mt][i] += sel[i];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) dp[mt][i] = acc[0][mt][i];
    }
  } else {
    // slot (kb, g) is row (kb/4)*16 + 4g + kb%4 of layer l: accumulator
    // dl[kb/4][kb%4] of this lane
    const int g = lane >> 4, c = lane & 15;
    const float* W[4];   // row 4g, by (mt ^ i) % 4: row 4g + i's column 16 mt + c but for constants
#pragma unroll
    for (int j = 0; j < 4; ++j) W[j] = reinterpret_cast<const float*>(wl) + f32_row(4 * g, H) + 16 * (j ^ g) + c;
    f32x4 acc[MTP];
    mfma_rows_f32<MTP, RT>(
        [&](int mt, int kq) {
          auto at = [&](int i) { return W[(mt ^ i) & 3][f32_rows(kq * 16, H) + f32_row(i, H) + (mt & ~3) * 16]; };
          return f32x4{at(0), at(1), at(2), at(3)};
        },
        [&](int kq, int i) { return dl[kq][i]; }, acc);
#pragma unroll
    for (int mt = 0; mt < MTP; ++mt)
#pragma unroll
      for (int i = 0; i < 4; ++i) dp[mt][i] = acc[mt][i];
  }
}

// BF16 staging of the weight gradient's operands, in two layouts. A lane's
// operand of a 32-vertex block is eight vertices (vb*32 + 8g ..) of one row,
// while its accumulators are four rows of one vertex.
//
// Staged<R>, [vertex][R rows]: the four rows are one 8-byte write, and gfx950's
// transposing LDS read (ds_read_b64_tr_b16: within 16 lanes, lane 4k + n holds
// columns 4n .. 4n + 3 of matrix row k, and lane r receives column r of the
// four rows) turns four vertices of 16 rows into half an operand: two reads an
// operand. Rows<SP>, [row][vertex]: one 16-byte read an operand, but a lane
// exchange, two byte permutes and three selects before a tile's writes. So
// deltas, which a wave reads for few row tiles, are staged by vertex; a
// layer's inputs by row where every wave reads all of their column tiles (the
// hidden-128 network all by vertex: 5.5 -> 6.4 ms per 2^22-sample step), by
// vertex where it reads one. Both by row before: hidden 64, 2^18 samples, K = 4
// 61 -> 58 us, K = 8 88 -> 82, K = 16 with selection 111.5 -> 107.5.
//
// Staged: vertex v of 32 sits in slot (v/4 % 2) 16 + (v/8) 4 + v % 4, so that a
// read of group g returns vertices 8g + 4t ..; rows are kept in units of 16.
// So that the eight slots of a half-wave's read, and the 16 of its write, cover
// the 64 banks, the units of a slot are permuted by key(slot) where R is a
// power of two (for an odd number of units the pitch itself spreads them), and
// the halves of a unit are swapped in the second 16 slots.
template <int R>
struct Staged {
  static constexpr int U = R / 16;
  static_assert(R % 16 == 0 && (U % 2 == 1 || U == 2 || U == 4 || U == 8), "rows of a staging buffer");
  __device__ __forceinline__ static int key(int slot) {
    return U == 8 ? (slot & 7) : (U == 4 ? ((slot >> 1) & 3) : (U == 2 ? ((slot >> 2) & 1) : 0));
  }
  // LDS address of unit u from that of unit 0 (buffers are 256-byte aligned)
  __device__ __forceinline__ static uint32_t unit(uint32_t base, int u) {
    return U % 2 ? base + u * 32 : base ^ (uint32_t)(u * 32);
  }
  // rows 4g .. 4g + 3 of unit 0 of vertex wave*16 + c
  __device__ __forceinline__ static uint32_t write_base(const void* buf, int wave, int g, int c) {
    const int v = (wave & 1) * 16 + c;
    const int slot = ((v >> 2) & 1) * 16 + (v >> 3) * 4 + (v & 3);
    return lds_addr(buf) + 2 * (((wave >> 1) * 32 + slot) * R + key(slot) * 16 + ((4 * g) ^ ((slot >> 4) * 8)));
  }
  // unit 0 of slot 4g + c/4, columns 4 (c % 4) ..: a lane's part of a transposing read
  __device__ __forceinline__ static uint32_t read_base(const void* buf, int g, int c) {
    const int slot = 4 * g + (c >> 2);
    return lds_addr(buf) + 2 * (slot * R + key(slot) * 16 + 4 * (c & 3));
  }
  __device__ __forceinline__ static bf16x8 operand(uint32_t base, int row, int vb) {
    typedef __attribute__((ext_vector_type(4))) short s16x4;
    typedef __attribute__((address_space(3))) s16x4* P;
    const uint32_t a = unit(base, row) + vb * 32 * R * 2;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((P)(uintptr_t)a);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((P)(uintptr_t)((a ^ 16) + 16 * R * 2));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  }
};

template <int SP>
struct Rows {
  __device__ __forceinline__ static uint32_t read_base(const void* buf, int g, int c) {
    return lds_addr(buf) + 2 * (c * SP + 8 * g);
  }
  __device__ __forceinline__ static bf16x8 operand(uint32_t base, int row, int vb) {
    return *(__attribute__((address_space(3))) bf16x8*)(uintptr_t)(base + 2 * (row * 16 * SP + vb * 32));
  }
};

// FP32 [row][vertex]: four vertices (vb*16 + 4g ..) an operand.
template <int SP>
struct RowsF32 {
  __device__ __forceinline__ static uint32_t read_base(const void* buf, int g, int c) {
    return lds_addr(buf) + 4 * (c * SP + 4 * g);
  }
  __device__ __forceinline__ static f32x4 operand(uint32_t base, int row, int vb) {
    return *(__attribute__((address_space(3))) f32x4*)(uintptr_t)(base + 4 * (row * 16 * SP + vb * 16));
  }
};

// One row tile into a Rows buffer at `tile` (its row 0, the wave's vertex
// column 0): lane (g, c) holds rows 4g..4g+3 of vertex c as two packed words,
// w0 (rows 4g, 4g+1) and w1 (rows 4g+2, 4g+3). Lanes c and c^1 (neighbouring
// vertices) swap half of them through one DPP move, so each writes two rows
// of both vertices as two 4-byte stores (the even lane rows 4g, 4g+1, the odd
// lane rows 4g+2, 4g+3; one ds_write2_b32) instead of four 2-byte stores.
template <int SP>
__device__ __forceinline__ void stage_tile_rows(__bf16* tile, uint32_t w0, uint32_t w1, int g, int c) {
  const bool odd = c & 1;
  const uint32_t send = odd ? w0 : w1;   // the rows the partner writes
  const uint32_t mine = odd ? w1 : w0;
  // quad_perm [1, 0, 3, 2]: the value of lane c^1
  const uint32_t recv = (uint32_t)__builtin_amdgcn_mov_dpp((int)send, 0xB1, 0xF, 0xF, false);
  // v_perm_b32 byte selectors over (recv: bytes 4..7, mine: bytes 0..3):
  // even lane (recv = vertex c+1) [mine.lo, recv.lo], [mine.hi, recv.hi];
  // odd lane (recv = vertex c-1) [recv.lo, mine.lo], [recv.hi, mine.hi]
  __bf16* const p = tile + (4 * g + (odd ? 2 : 0)) * SP + (c & ~1);
  *reinterpret_cast<uint32_t*>(p) = __builtin_amdgcn_perm(recv, mine, odd ? 0x01000504u : 0x05040100u);
  *reinterpret_cast<uint32_t*>(p + SP) = __builtin_amdgcn_perm(recv, mine, odd ? 0x03020706u : 0x07060302u);
}
template <int SP, int RT>
__device__ __forceinline__ void stage_words_rows(__bf16* buf, const uint32_t (&w)[RT][2], int wave, int lane) {
#pragma unroll
  for (int mt = 0; mt < RT; ++mt)
    stage_tile_rows<SP>(buf + mt * 16 * SP + wave * 16, w[mt][0], w[mt][1], lane >> 4, lane & 15);
}

// Packed rows (words) of a wave's 16-vertex block into a Staged buffer.
template <int R, int RT>
__device__ __forceinline__ void stage_words(void* buf, const uint32_t (&w)[RT][2], int wave, int lane) {
  static_assert(RT * 16 <= R, "the buffer holds the rows");
  typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
  const uint32_t base = Staged<R>::write_base(buf, wave, lane >> 4, lane & 15);
#pragma unroll
  for (int mt = 0; mt < RT; ++mt)
    *(__attribute__((address_space(3))) u32x2*)(uintptr_t)Staged<R>::unit(base, mt) = u32x2{w[mt][0], w[mt][1]};
}

// Layer 0's BF16 input (the values the forward used) into a staging buffer of
// R = 16 rows (raw: lane group g holds rows 4g ..) or 64 (encoded: rows
// kb*32 + 8g .. + 7).
__device__ __forceinline__ void stage_input_bf16(void* buf, const bf16x4& x, int wave, int lane) {
  *(__attribute__((address_space(3))) bf16x4*)(uintptr_t)Staged<16>::write_base(buf, wave, lane >> 4, lane & 15) = x;
}
__device__ __forceinline__ void stage_input_bf16(void* buf, const EncodedInput& x, int wave, int lane) {
  const int g = lane >> 4, c = lane & 15;
  // lane groups 2u, 2u + 1 hold the halves of unit u
  const uint32_t base = Staged<64>::write_base(buf, wave, 2 * (g & 1), c);
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
    *(__attribute__((address_space(3))) bf16x8*)(uintptr_t)Staged<64>::unit(base, 2 * kb + (g >> 1)) = x.b[kb];
}

// Write a wave's accumulator-layout block [RT*16 rows][16 vertices] into the
// FP32 staging buffer [row][vertex] at vertex columns wave*16 .. (stage_col_f32).
template <int RT, int SP>
__device__ __forceinline__ void stage_rows_f32(float* buf, const float (&x)[RT][4], int wave, int lane) {
  const int g = lane >> 4, col = wave * 16 + stage_col_f32(lane & 15);
#pragma unroll
  for (int mt = 0; mt < RT; ++mt)
#pragma unroll
    for (int i = 0; i < 4; ++i) buf[(mt * 16 + 4 * g + i) * SP + col] = x[mt][i];
}

// BF16 rows of a block packed in pairs (as the MFMA operands hold them):
// w[mt][0] = rows mt*16 + 4g, + 4g + 1 and w[mt][1] = rows + 4g + 2, + 4g + 3
// of vertex c, low half first; rounded to nearest even.
template <int RT>
__device__ __forceinline__ void pack_rows(const float (&x)[RT][4], uint32_t (&w)[RT][2]) {
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  typedef __attribute__((ext_vector_type(2))) float f32x2;
#pragma unroll
  for (int mt = 0; mt < RT; ++mt)
#pragma unroll
    for (int k = 0; k < 2; ++k)
      w[mt][k] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){x[mt][2 * k], x[mt][2 * k + 1]}, bf16x2));
}

// d *= (h != 0) per BF16 half: the ReLU derivative, h being packed ReLU
// outputs (non-negative, so min(h, 1) as a 16-bit integer is the indicator)
template <int RT>
__device__ __forceinline__ void mask_rows(uint32_t (&d)[RT][2], const uint32_t (&h)[RT][2]) {
  typedef __attribute__((ext_vector_type(2))) unsigned short u16x2;
#pragma unroll
  for (int mt = 0; mt < RT; ++mt)
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const u16x2 ind = __builtin_bit_cast(u16x2, relu_indicator(h[mt][k]));
      d[mt][k] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, d[mt][k]) * ind);
    }
}

// dgrad (BF16) with the deltas already packed: the packed words are the B
// operands as they are (an even number of row tiles, no selection tile).
template <int H, int RT>
__device__ __forceinline__ void dgrad_words(const void* wl, const uint32_t (&dw)[RT][2], float (&dp)[H / 16][4],
                                            int lane) {
  static_assert(RT % 2 == 0, "whole 32-wide blocks");
  constexpr int MTP = H / 16, KB = RT / 2;
  typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_;
  bf16x8 b[KB];
#pragma unroll
  for (int kb = 0; kb < KB; ++kb)
    b[kb] = __builtin_bit_cast(bf16x8, u32x4_{dw[2 * kb][0], dw[2 * kb][1], dw[2 * kb + 1][0], dw[2 * kb + 1][1]});
  f32x4 acc[1][MTP];
  mfma_rows<MTP, KB, 1>(reinterpret_cast<const bf16x8*>(wl), [&](int, int kb) { return b[kb]; }, acc, lane);
#pragma unroll
  for (int mt = 0; mt < MTP; ++mt)
#pragma unroll
    for (int i = 0; i < 4; ++i) dp[mt][i] = acc[0][mt][i];
}

// acc[r][ct] += D[rows (r0+r)*16..][v] * Hs[cols (c0+ct)*16..][v]^T over the
// NV vertices staged in BF16 in the layouts DL and HL
template <typename DL, typename HL, int NV, int NR, int NC>
__device__ __forceinline__ void wgrad_block(const void* dst, const void* hst, int r0, int c0, f32x4 (&acc)[NR][NC],
                                            int lane) {
  asm volatile("" : "+v"(lane));   // addresses formed here, not kept across the kernel
  const int g = lane >> 4, c = lane & 15;
  const uint32_t db = DL::read_base(dst, g, c), hb = HL::read_base(hst, g, c);
#pragma unroll
  for (int vb = 0; vb < NV / 32; ++vb) {
    bf16x8 h[NC], d[NR];
#pragma unroll
    for (int ct = 0; ct < NC; ++ct) h[ct] = HL::operand(hb, c0 + ct, vb);
#pragma unroll
    for (int r = 0; r < NR; ++r) d[r] = DL::operand(db, r0 + r, vb);
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int ct = 0; ct < NC; ++ct) acc[r][ct] = mfma_bf16_32(d[r], h[ct], acc[r][ct]);
  }
}

template <int NR, int NC>
__device__ __forceinline__ void zero_tiles(f32x4 (&acc)[NR][NC]) {
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int ct = 0; ct < NC; ++ct) acc[r][ct] = zero4();
}

// The same for all column tiles and a wave's row tiles in FP32 ([row][vertex],
// pitch SP).
template <int SP, int NR, int NC, int NV = kWGV>
__device__ __forceinline__ void wgrad_tiles_f32(const float* dst, const float* hst, const int (&rt)[NR], int nrt,
                                                f32x4 (&acc)[NR][NC], int lane) {
  const int g = lane >> 4, c = lane & 15;
  // lane group g takes columns vb*16 + 4g .. + 3, one 16-byte read per row
#pragma unroll
  for (int vb = 0; vb < NV / 16; ++vb) {
    f32x4 hb[NC];
#pragma unroll
    for (int ct = 0; ct < NC; ++ct)
      hb[ct] = *reinterpret_cast<const f32x4*>(hst + (ct * 16 + c) * SP + vb * 16 + 4 * g);
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      if (r < nrt) {
        const f32x4 da = *reinterpret_cast<const f32x4*>(dst + (rt[r] * 16 + c) * SP + vb * 16 + 4 * g);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int ct = 0; ct < NC; ++ct) acc[r][ct] = mfma_f32_4(da[i], hb[ct][i], acc[r][ct]);
      }
    }
  }
}

// Ownership of a layer's dW tiles (RT row tiles x CT column tiles) among the
// NW waves of a workgroup, tile j of a wave being (rt(w, j), ct(w, j)):
// * RT a multiple of NW (row mode): wave w owns row tiles w, w + NW, ... and
//   every column tile (per staged block: CT column operands, one row operand
//   per row tile);
// * otherwise (column mode, NW a multiple of CT): wave w owns column tile
//   w % CT and row tiles w / CT + (NW / CT) j below RT (one column operand,
//   one row operand per tile), so that an odd row tile (the selection
//   output's) adds one tile to some waves rather than CT to one.
template <int RT, int CT, int NW>
struct Own {
  static constexpr bool ROW = RT >= NW && RT % NW == 0;
  static_assert(ROW || NW % CT == 0, "waves must split evenly over the column tiles");
  static constexpr int STEP = ROW ? NW : NW / CT;
  static constexpr int NRW = (RT + STEP - 1) / STEP;        // row tiles per wave
  static constexpr int TPW = ROW ? NRW * CT : NRW;          // tiles per wave
  __device__ __forceinline__ static int rt(int wave, int j) { return ROW ? wave + NW * (j / CT) : wave / CT + STEP * j; }
  __device__ __forceinline__ static int ct(int wave, int j) { return ROW ? j % CT : wave % CT; }
};

// acc[j] += D[rows of rt(j)][v] * Hs[cols of ct(j)][v]^T over NV staged
// vertices, in the layouts DL and HL. The operands of vertex block vb + 1 are
// read while block vb is multiplied (two register sets), so the LDS latency
// overlaps the MFMAs.
template <int PREC, typename DL, typename HL, int RT, int CT, int NW, int NV>
__device__ __forceinline__ void wgrad_own(const void* dst, const void* hst, f32x4 (&acc)[Own<RT, CT, NW>::TPW],
                                          int wave, int lane) {
  typedef Own<RT, CT, NW> O;
  typedef decltype(DL::operand(0, 0, 0)) Op;
  const int g = lane >> 4, c = lane & 15;
  constexpr int VB = PREC == 1 ? NV / 32 : NV / 16;
  constexpr int NH_ = O::ROW ? CT : 1, ND = O::ROW ? O::NRW : O::TPW;
  const uint32_t db = DL::read_base(dst, g, c), hb = HL::read_base(hst, g, c);
  auto d_op = [&](int row, int vb) { return DL::operand(db, row, vb); };
  auto h_op = [&](int row, int vb) { return HL::operand(hb, row, vb); };
  struct Ops { Op h[NH_]; Op d[ND]; };
  auto load = [&](int vb, Ops& o) {
    if constexpr (O::ROW) {
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) o.h[ct] = h_op(ct, vb);
#pragma unroll
      for (int r = 0; r < O::NRW; ++r)
        if (O::rt(wave, r * CT) < RT) o.d[r] = d_op(O::rt(wave, r * CT), vb);
    } else {
      o.h[0] = h_op(O::ct(wave, 0), vb);
#pragma unroll
      for (int j = 0; j < O::TPW; ++j)
        if (O::rt(wave, j) < RT) o.d[j] = d_op(O::rt(wave, j), vb);
    }
  };
  Ops ops[2];
  load(0, ops[0]);
#pragma unroll
  for (int vb = 0; vb < VB; ++vb) {
    if (vb + 1 < VB) load(vb + 1, ops[(vb + 1) & 1]);
    const Ops& o = ops[vb & 1];
    constexpr int NI = PREC == 1 ? 1 : 4;   // contraction steps of a block
#pragma unroll
    for (int i = 0; i < NI; ++i) {
#pragma unroll
      for (int j = 0; j < O::TPW; ++j) {
        const int r = O::ROW ? j / CT : j, ct = O::ROW ? j % CT : 0;
        if (O::rt(wave, j) < RT) {
          if constexpr (PREC == 1) acc[j] = mfma_bf16_32(o.d[r], o.h[ct], acc[j]);
          else acc[j] = mfma_f32_4(o.d[r][i], o.h[ct][i], acc[j]);
        }
      }
    }
  }
}

// Flush a wave's owned dW tiles of layer l to the workgroup's canonical partial.
template <int RT, int CT, int NW>
__device__ __forceinline__ void flush_own(float* part, const NetDims& d, int l,
                                          const f32x4 (&acc)[Own<RT, CT, NW>::TPW], int wave, int lane) {
  typedef Own<RT, CT, NW> O;
  const int g = lane >> 4, c = lane & 15;
  const int cols = d.cols(l);
  const int64_t off = d.canon_off(l);
#pragma unroll
  for (int j = 0; j < O::TPW; ++j) {
    const int k = O::ct(wave, j) * 16 + c;
    if (O::rt(wave, j) >= RT || k >= cols) continue;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int R = O::rt(wave, j) * 16 + 4 * g + i;
      const int n = (l == d.NH) ? canon_out_row(R, d.K) : R;
      if (n >= 0) part[off + (int64_t)n * cols + k] = acc[j][i];   // n < 0: padding rows
    }
  }
}

// Flush a wave's dW tiles of layer l to the workgroup's canonical partial.
// PAD: the tiles may hold the selection tile's padding rows (skipped).
template <int NR, int NC, bool PAD = false>
__device__ __forceinline__ void flush_tiles(float* part, const NetDims& d, int l, const int (&rt)[NR], int nrt,
                                            const f32x4 (&acc)[NR][NC], int lane, int c0 = 0) {
  const int g = lane >> 4, c = lane & 15;
  const int cols = d.cols(l);
  const int64_t off = d.canon_off(l);
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    if (r >= nrt) continue;
#pragma unroll
    for (int ct = 0; ct < NC; ++ct) {
      const int k = (c0 + ct) * 16 + c;
      if (k >= cols) continue;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int R = rt[r] * 16 + 4 * g + i;
        const int n = (l == d.NH) ? canon_out_row(R, d.K) : R;
        if (!PAD || n >= 0) part[off + (int64_t)n * cols + k] = acc[r][ct][i];   // n < 0: padding rows
      }
    }
  }
}

// The same for a block of tiles (wgrad_block's).
template <bool PAD, int NR, int NC>
__device__ __forceinline__ void flush_block(float* part, const NetDims& d, int l, int r0, int c0,
                                            const f32x4 (&acc)[NR][NC], int lane) {
  int rt[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) rt[r] = r0 + r;
  flush_tiles<NR, NC, PAD>(part, d, l, rt, NR, acc, lane, c0);
}

}  // namespace nasg
