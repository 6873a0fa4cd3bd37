// Per-vertex NASG epilogues on the MLP's output accumulators.
//
// `out[mt][i]` at lane (g, c) is raw output t = mt*4 + i of lobe
// g*KQ + t % KQ, parameter t / KQ (layout.hpp), for vertex c. Each lane
// handles KQ = K/4 lobes of one vertex; the four lanes c, c+16, c+32, c+48
// together hold the K lobes.
#pragma once

#include "kernels.hpp"

namespace nasg {

template <int KQ, int MTO>
__device__ __forceinline__ void lobe_raw(const float (&out)[MTO][4], int q, float o[8]) {
#pragma unroll
  for (int p = 0; p < 8; ++p) {
    const int t = p * KQ + q;
    o[p] = out[t >> 2][t & 3];
  }
}

// Weighted NLL of one vertex and its gradient w.r.t. the raw outputs
// (Sec. 4.2): gs = dL/dlog q = -w/B (0 for padding lanes). Writes dl in the
// accumulator layout and returns the vertex's log term (log q; with the
// selection output, e log q_hat + (1 - e) log q).
//
// One pass over the lobes: each lobe is decoded and evaluated once, and its
// log-density's partials d ell_k / d o_p (p < 7) go straight into dl. They
// are linear in the upstream factor, which is only known once log q is:
// dL/d o_p = gq r_k d ell_k / d o_p with r_k = q_k / q, and for the logit
// dL/d o_7 = gq (r_k - A_k) (through the softmax). A second, cheap loop
// scales them.
//
// S = 1 (selection output, the blended loss of Sec. 4.2): with c the
// sigmoid of the selection logit (output row 8K, held by lane group 0) and
// q_hat = c q + (1 - c) p_fs, the loss term e log q_hat + (1 - e) log q has
// d/dlog q = e c q / q_hat + (1 - e), so gq = gs times that, and
// d/dz (z the selection logit) = e (q - p_fs) c (1 - c) / q_hat.
template <int KQ, int MTO, int S = 0>
__device__ __forceinline__ float train_epilogue(const float (&out)[MTO][4], float vx, float vy, float vz,
                                                float gs, bool valid, float eps, float (&dl)[MTO][4],
                                                float pdf_bsdf = 0.0f, float mis_e = 0.0f, float amul = 1.0f) {
  constexpr int TS = 2 * KQ;   // the selection tile (S = 1)
  static_assert(MTO == 2 * KQ + S, "output tiles: 8K rows plus the selection tile");
  // softmax of the K logits: A_k = e^{alpha_k - m} / sum, kept for the logit gradient
  float ea[KQ];
  float lse, inv_se;
  {
    float mx = -INFINITY;
#pragma unroll
    for (int q = 0; q < KQ; ++q) {
      const int t = 7 * KQ + q;
      mx = fmaxf(mx, out[t >> 2][t & 3]);
    }
    mx = xchg_max(mx);
    float se = 0.0f;
#pragma unroll
    for (int q = 0; q < KQ; ++q) {
      const int t = 7 * KQ + q;
      ea[q] = fexp_sub(out[t >> 2][t & 3], mx);
      se += ea[q];
    }
    se = xchg_sum(se);
    lse = mx + flog(se);
    inv_se = frcp(se);
  }
  float ell[KQ];
#pragma unroll
  for (int q = 0; q < KQ; ++q) {
    float o[8];
    lobe_raw<KQ, MTO>(out, q, o);
    Lobe L;
    LobeAux X;
    decode_lobe(o, eps, L, X, amul);
    L.logc = (o[7] - lse) - X.logK;
    const Eval e = eval_lobe(L, vx, vy, vz, eps);
    ell[q] = e.ell;
    float gq[8];
    backward_lobe(L, X, e, vx, vy, vz, eps, 1.0f, 0.0f, gq);
#pragma unroll
    for (int p = 0; p < 7; ++p) {
      const int t = p * KQ + q;
      dl[t >> 2][t & 3] = gq[p];
    }
  }
  const float logq = mixture_lse<KQ>(ell);
  float lterm = logq, gsq = gs;
  if constexpr (S == 1) {
    const int c = lane_id() & 15;
    const float z = __shfl(out[TS][0], c);   // lane (0, c) holds row 8K of vertex c
    const float cs = frcp(1.0f + fexp(-z));
    const float qv = fexp(logq);
    const float qh = fmaf(cs, qv - pdf_bsdf, pdf_bsdf);   // c q + (1 - c) p_fs
    const float iqh = frcp(qh);
    lterm = fmaf(mis_e, flog(qh), (1.0f - mis_e) * logq);
    gsq = gs * fmaf(mis_e * cs, qv * iqh, 1.0f - mis_e);
    const float gz = gs * mis_e * (qv - pdf_bsdf) * cs * (1.0f - cs) * iqh;
    const bool g0 = lane_id() < 16;
#pragma unroll
    for (int i = 0; i < 4; ++i) dl[TS][i] = (g0 && i == 0) ? gz : 0.0f;
  }
#pragma unroll
  for (int q = 0; q < KQ; ++q) {
    const int t7 = 7 * KQ + q;
    const float r = valid ? fexp_sub(ell[q], logq) : 0.0f;
    const float Aq = ea[q] * inv_se;
    const float sc = gsq * r;
#pragma unroll
    for (int p = 0; p < 7; ++p) {
      const int t = p * KQ + q;
      dl[t >> 2][t & 3] *= sc;
    }
    dl[t7 >> 2][t7 & 3] = gsq * (r - Aq);
  }
  // padding lanes (a branch taken only in a batch's last tile): zeroed
  // outright, so that no non-finite partial of their arbitrary lobes reaches
  // the weight gradient as 0 * inf
  if (!valid) {
#pragma unroll
    for (int mt = 0; mt < MTO; ++mt)
#pragma unroll
      for (int i = 0; i < 4; ++i) dl[mt][i] = 0.0f;
  }
  return lterm;
}

// A query's decode of one vertex's lobes (Tab. "decoding") into lb; the
// mixture weights (softmax of the K logits) are A_k = ea_k inv_se; returns the
// logits' log-sum-exp.
template <int KQ, int MTO>
__device__ __forceinline__ float query_decode(const float (&out)[MTO][4], float eps, QueryLobe (&lb)[KQ],
                                              float (&ea)[KQ], float& inv_se, float abias) {
#pragma clang fp contract(off)
  float alpha[KQ];
#pragma unroll
  for (int q = 0; q < KQ; ++q) {
    float o[8];
    lobe_raw<KQ, MTO>(out, q, o);
    decode_lobe_query(o, eps, lb[q], abias);
    alpha[q] = o[7];
  }
  // mixture weights: softmax over the K logits
  float mx = alpha[0];
#pragma unroll
  for (int q = 1; q < KQ; ++q) mx = fmaxf(mx, alpha[q]);
  mx = quad_max(mx);
  float se = 0.0f;
#pragma unroll
  for (int q = 0; q < KQ; ++q) {
    ea[q] = fexp_sub(alpha[q], mx);
    se += ea[q];
  }
  se = quad_sum(se);
  inv_se = frcp(se);
#pragma unroll
  for (int q = 0; q < KQ; ++q) lb[q].c *= ea[q] * inv_se;
  // where the rounding of logits beyond about 1e9 overflows the sum, the
  // log-sum-exp is +infinity, every log c_k of the records -infinity and the
  // density 0; here 0 times infinity
  if (__any(se == INFINITY)) {
#pragma unroll
    for (int q = 0; q < KQ; ++q) lb[q].c = fsel(se == INFINITY, 0.0f, lb[q].c);
  }
  return mx + flog(se);
}

// One App. C sample from a query lobe, normalised to unit length.
__device__ __forceinline__ void sample_unit(const QueryLobe& s, float xi0, float xi1, float xi2, float eps, float& vx,
                                            float& vy, float& vz) {
  const Lobe L = {s.zx, s.zy, s.zz, s.xx, s.xy, s.xz, s.lam, s.a, 0.0f};
  sample_lobe(L, xi0, xi1, xi2, eps, vx, vy, vz);
  const float inv = frsq(fmaf(vx, vx, fmaf(vy, vy, vz * vz)));
  vx *= inv;
  vy *= inv;
  vz *= inv;
}

// sum_k c_k G_k at a unit direction (the mixture pdf is query_pdf_scale times
// it), over the lane's lobes, then the vertex's 4 lanes. No running maximum is
// needed where the sum is above 2^-64: a G beneath the float range (2^-126)
// loses less than c_k 2^-126 there, and c_k is at most 2^33 at the clamps of
// lambda and a (and epsilon not above a's). The lobe that the direction was drawn from usually sees to
// that (A_k and G of about 2^-24 at least, for 24-bit uniforms), but not where
// xi_sel = 0 picked a lobe of any weight, or xi0 = 0 the antipode, where G = 0:
// a wave with such a vertex takes its sum by the logarithm.
constexpr float kLinearSumMin = 5.421010862427522e-20f;   // 2^-64
template <int KQ>
__device__ __forceinline__ float query_sum(const QueryLobe (&lb)[KQ], float vx, float vy, float vz, float eps) {
#pragma clang fp contract(off)
  float s = 0.0f;
#pragma unroll
  for (int q = 0; q < KQ; ++q) {
    bool on;
    const float lg = eval_query_lobe(lb[q], vx, vy, vz, eps, on);
    // a lobe without density adds nothing, whatever its weight (NaN among them)
    s = fsel(on, fmaf(lb[q].c, __builtin_amdgcn_exp2f(lg), s), s);
  }
  return quad_sum(s);
}
template <int KQ>
__device__ __forceinline__ float query_sum_log(const QueryLobe (&lb)[KQ], float vx, float vy, float vz, float eps) {
#pragma clang fp contract(off)
  float t[KQ], m = -INFINITY, e = 0.0f;
#pragma unroll
  for (int q = 0; q < KQ; ++q) {
    bool on;
    const float lg = eval_query_lobe(lb[q], vx, vy, vz, eps, on);
    t[q] = fsel(on, flog2(lb[q].c) + lg, -INFINITY);
    m = fmaxf(m, t[q]);
  }
  m = quad_max(m);
#pragma unroll
  for (int q = 0; q < KQ; ++q) e += __builtin_amdgcn_exp2f(t[q] - m);
  e = quad_sum(e);
  return fsel(m == -INFINITY, 0.0f, __builtin_amdgcn_exp2f(m + flog2(e)));
}

// Records of one 16-vertex block's lobes (optional output of a query); lse:
// the logits' log-sum-exp.
template <int KQ, int MTO>
__device__ __forceinline__ void store_records(float* rec_out, const float (&out)[MTO][4], const QueryLobe (&lb)[KQ],
                                              float lse, float eps, int64_t v, int g) {
  constexpr int K = 4 * KQ;
  float* base = rec_out + (v / kRecTile) * 9 * K * kRecTile + g * KQ * kRecTile + (v % kRecTile);
  // opaque to the compiler, which otherwise keeps an address per parameter
  // live across the whole batch loop (registers that the K = 16 kernel spills)
  asm("" : "+v"(base));
#pragma unroll
  for (int q = 0; q < KQ; ++q) {
    float o[8];
    lobe_raw<KQ, MTO>(out, q, o);
    const QueryLobe& L = lb[q];
    const float loglam = fminf(fmaxf(o[5], -kLogClamp), kLogClamp);
    const float lam = fexp(loglam);
    // one lobe at a time: mixed by the scheduler, the K = 16 kernel spills
    __builtin_amdgcn_sched_barrier(0);
    const float logc = (o[7] - lse) - log_normaliser(lam, loglam, L.a, eps);
    const float vals[9] = {L.zx, L.zy, L.zz, L.xx, L.xy, L.xz, L.lam, L.a, logc};
#pragma unroll
    for (int p = 0; p < 9; ++p) base[(p * K + q) * kRecTile] = vals[p];
  }
}

// Guiding queries of NBLK 16-vertex blocks (vertices v0 + 16 b + c): decode,
// inverse-CDF lobe choice, App. C sample, mixture pdf at the sample, stores.
// block(b, out) writes block b's raw outputs; xi(r, i) returns uniform row r
// of vertex v0 + i. Lane (g, c) holds lobes g*KQ .. of vertex c of every
// block and samples one vertex, c of block g % NBLK: the chosen lobe of each
// block moves to the lanes that sample it, and the directions go back to the
// lanes that hold the block's lobes. Per vertex, the same operations in the
// same order for every NBLK, so the same results bit for bit. SPLIT keeps the
// next block's forward out of a block's decode.
template <int KQ, int S, int NBLK, bool REC, bool SPLIT, int MTO, typename BlockFn, typename XiFn>
__device__ __forceinline__ void query_epilogue(const QueryArgs& a, int64_t v0, int lane, BlockFn block, XiFn xi) {
  static_assert(NBLK == 1 || NBLK == 2 || NBLK == 4, "lane groups share the blocks evenly");
  const int g = lane >> 4, c = lane & 15;
  const int i = (g % NBLK) * kTileV + c;   // the vertex this lane samples
  const int64_t vi = v0 + i;
  const bool vi_valid = vi < a.B;
  // one block per pass: its uniforms, in registers (query_kernel) or requested
  // from global memory here (the streamed kernels) and used after the lobes are
  // decoded; the other forms' are staged in LDS
  float xr[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  if (NBLK == 1 && vi_valid) {
#pragma unroll
    for (int r = 0; r < 4; ++r) xr[r] = xi(r, i);
  }
  QueryLobe lb[NBLK][KQ];
  QueryLobe ch = {};
  const float abias = a.amul > 0.0f ? 0.0f : -INFINITY;   // log2 of the anisotropy's factor
#pragma unroll
  for (int b = 0; b < NBLK; ++b) {
    const int64_t v = v0 + b * kTileV + c;
    const bool valid = v < a.B;
    float out[MTO][4];
    // a wave in its forward goes first: its MFMAs and LDS reads then run beside
    // the VALU work of the SIMD's other wave, whose instructions fill the gaps
    // (2^20 vertices: K = 16 134.7 -> 132.6 us, K = 8 90.3 -> 88.3, K = 4 55.2 ->
    // 53.8; FP32 K = 16 at 2^19 211 -> 208; the other way round K = 16 136.8).
    // In the hidden-64 networks only: the hidden-128 kernels have run the forward
    // before, and block(b, out) copies its registers
    __builtin_amdgcn_s_setprio(1);
    block(b, out);
    __builtin_amdgcn_s_setprio(0);
    float ea[KQ], inv_se;
    const float lse = query_decode<KQ, MTO>(out, a.eps, lb[b], ea, inv_se, abias);
    const float xs = NBLK == 1 ? xr[0] : (valid ? xi(0, b * kTileV + c) : 0.0f);
    const int k = select_lobe<KQ>(ea, inv_se, xs, g, c);
    const QueryLobe r = broadcast_lobe<KQ>(lb[b], k, c);
    if (NBLK == 1 || g % NBLK == b) ch = r;
    // selection probability c = sigmoid(o[8K]) (Tab. "decoding")
    if (S == 1 && a.sel_out != nullptr && valid && g == 0) a.sel_out[v] = frcp(1.0f + fexp(-out[MTO - 1][0]));
    if (REC && valid) store_records<KQ, MTO>(a.rec_out, out, lb[b], lse, a.eps, v, g);
    if constexpr (SPLIT) __builtin_amdgcn_sched_barrier(0);
  }
  if (NBLK > 1 && vi_valid) {
#pragma unroll
    for (int r = 1; r < 4; ++r) xr[r] = xi(r, i);
  }
  float vx, vy, vz;
  sample_unit(ch, xr[1], xr[2], xr[3], a.eps, vx, vy, vz);
  // block b's directions, at the lanes that hold its lobes
  auto at_block = [&](int b, float& bx, float& by, float& bz) {
    bx = vx;
    by = vy;
    bz = vz;
    if constexpr (NBLK > 1) {
      const int src = b * kTileV + c;
      bx = __shfl(vx, src);
      by = __shfl(vy, src);
      bz = __shfl(vz, src);
    }
  };
  float sum = 0.0f;
#pragma unroll
  for (int b = 0; b < NBLK; ++b) {
    float bx, by, bz;
    at_block(b, bx, by, bz);
    const float s = query_sum<KQ>(lb[b], bx, by, bz, a.eps);
    if (NBLK == 1 || g % NBLK == b) sum = s;
  }
  if (__any(sum < kLinearSumMin)) {
    float logsum = 0.0f;
#pragma unroll
    for (int b = 0; b < NBLK; ++b) {
      float bx, by, bz;
      at_block(b, bx, by, bz);
      const float s = query_sum_log<KQ>(lb[b], bx, by, bz, a.eps);
      if (NBLK == 1 || g % NBLK == b) logsum = s;
    }
    sum = fsel(sum < kLinearSumMin, logsum, sum);
  }
  const float pdf = sum * query_pdf_scale(a.eps);
  if (vi_valid && g < NBLK) {
    a.dir_out[vi] = vx;
    a.dir_out[a.ld + vi] = vy;
    a.dir_out[2 * a.ld + vi] = vz;
    a.pdf_out[vi] = pdf;
  }
}

}  // namespace nasg
