// Matched correction pass (Sec. 3.4; App. B.6.3 "Matched correction").
//
// delta_i = (sum_j P_ij dP_ij) / (sum_j P_ij) with the FP32 probabilities
// P = 2^(tau log2e (S - LSE / tau)) recomputed from the FP8 scores, and
// dP = dO_row V_row^T (MX MFMA, FP32).  Sums of P dP and of P are formed in
// FP32 over each aligned 32-key group, the group sums are accumulated in
// FP64, and delta is stored as an FP32 pair (hi, lo) with hi + lo the FP64
// quotient to about 2^-48.  Dividing by sum P makes the pair the exact
// centring constant of the P the backward recomputes, even where the stored
// LSE leaves sum P a few ulp away from 1.  Compensated variant (COMP): every
// product P dP is formed exactly in FP64 and all sums run in FP64, so delta
// carries no FP32 rounding of the terms it cancels.
//
// Workgroup: NW waves x 32 or 64 queries of one (batch, query head); 128-key
// tiles (64 at 192 / 128) of K and V (row copies) reach LDS by direct loads,
// double-buffered, so the next tile streams in while the current one is
// computed.  S^T and dP^T put one query in each lane (row reductions in-lane
// plus one exchange with lane l ^ 32).  The isolated score channel (if any)
// is zeroed in the Q operand; its product and the shift -LSE / tau are added
// to the scores by one FP32 rank-2 MFMA.  P and dP use exactly the
// operations of the backward kernel (same MX MFMA products and k order, the
// same rank-2 update, bwd_prob()), so the backward's dS = P (dP - delta) sums
// to zero over every row up to FP32 rounding of its own terms.  Only the 32-key group holding the
// diagonal is masked; groups in a wave's future (causal) or past the last key
// are skipped.
#include <type_traits>

#include "common.hpp"
#include "dma.hpp"
#include "kernels.hpp"
#include "tiles.hpp"

namespace afp8 {

// QB: 32-query blocks per wave (2: every K / V fragment read from LDS serves
// two blocks).
template <int DQK, int DV, int NH = 1, int QB_ = 1>
struct DeltaCfg {
  // 192 / 128 heads take 64-key tiles, so that two double-buffered workgroups
  // fit a CU; dv = 256 keeps 128-key tiles and one workgroup, since two do not
  // fit its registers.
  static constexpr bool WIDE = DQK + DV > 256;
  static constexpr int QB = QB_;
  static constexpr int NW = 4, NT = 64 * NW, BQ = 32 * NW * QB, BK = WIDE && DV <= 128 ? 64 : 128;
  static constexpr int al16(int x) { return (x + 15) & ~15; }
  static constexpr int K_OFF = 0;                               // K row codes [BK][DQK], swizzled
  static constexpr int V_OFF = K_OFF + BK * DQK;                // V row codes [BK][DV], swizzled
  static constexpr int KS_OFF = V_OFF + BK * DV;                // K row scales [BK][DQK/32]
  static constexpr int VS_OFF = al16(KS_OFF + BK * DQK / 32);   // V row scales [BK][DV/32]
  // FP32 A operands of the rank-2 updates, [BK] each: the isolated channel's
  // key values, ones (NH = 3: then channels 1 and 2)
  static constexpr int KH_OFF = al16(VS_OFF + BK * DV / 32);
  static constexpr int NKH = NH == 3 ? 4 : 2;
  static constexpr int STAGE = KH_OFF + BK * 4 * NKH;
  // two workgroups per CU where both stage buffers fit 80 KB
  static constexpr int WGS = 2 * STAGE <= 80 * 1024 ? 2 : 1;
};

// A wave's work is a sequence of units (32-key group, 32-query block).  The
// MFMAs of one unit are interleaved with the vector work of the unit before
// it, one MFMA at a time with its share of that work behind it: a wave issues
// in order, so vector work placed after a run of MFMAs waits until the last
// of them has issued, 64 cycles each (measured: one 32x32x64 MFMA with 16
// vector instructions behind it takes 86 cycles with two waves per SIMD, 64
// and 84 apart).  On 4 x 8192 tokens, 16 / 4 heads of 128, causal: 0.674 ms
// with each unit's five MFMAs in a row, 0.618 interleaved, 0.556 with two
// blocks per wave; 600 cycles a unit, of which the MFMA pipe is busy 320 and
// vector issue 400.  The LDS operands of a fragment are read again right after
// its last MFMA, a unit ahead of their use, across tiles as well: the barrier
// of a tile comes before its last unit, whose operands are in registers by
// then.

// CAUSAL: the mask (key length = query length) or every key of Nk; COMP:
// FP64 products and sums; NH: isolated score channels (with 3, channels 1
// and 2 take a second rank-2 FP32 MFMA, the first shares one with the shift)
template <int DQK, int DV, bool CAUSAL, bool COMP, int NH, int QB>
__global__ __launch_bounds__(256, (DeltaCfg<DQK, DV, NH, QB>::WGS)) void delta_matching_kernel(AttnArgs a) {
  using C = DeltaCfg<DQK, DV, NH, QB>;
  constexpr int NW = C::NW, BQ = C::BQ, BK = C::BK, NG = BK / 32;
  constexpr int KS = DQK / 64, VS = DV / 64;
  __shared__ __attribute__((aligned(16))) uint8_t stA[C::STAGE];
  __shared__ __attribute__((aligned(16))) uint8_t stB[C::STAGE];
  __shared__ int hot_slot[NH];

  const int lane = threadIdx.x & 63, w = wave_id(), hf = lane >> 5, li = lane & 31;
  constexpr bool causal = CAUSAL;
  const int N = (int)a.N, Nk = CAUSAL ? N : (int)a.Nk;
  const int nqb = (N + BQ - 1) / BQ;
  const WgCoord wc = query_major_coord((int)blockIdx.x, (int)a.B, (int)a.Hq, (int)a.Hkv, a.lens_q != nullptr);
  const int qb = nqb - 1 - wc.r;              // longest causal rows first
  const int h = wc.h, b = wc.b, kh = h / (int)a.G;
  // the sequence's own lengths bound the work; N and Nk remain the strides
  const SeqLens L = seq_lens<CAUSAL>(a, b, N, Nk);
  if (qb * BQ >= L.q) return;                 // the whole block is past the sequence
  const int q0 = qb * BQ + 32 * QB * w;       // the wave's first query
  const bool live = q0 < L.q;
  int hots[NH];
  if constexpr (NH == 1) hots[0] = select_hot_channel<DQK>(a.q_amax, a.k_amax, b, kh, a.Hq, a.Hkv, a.G, hot_slot);
  else select_hot_channels<DQK, NH>(a.q_amax, a.k_amax, b, kh, a.Hq, a.Hkv, a.G, hot_slot, hots);
  const int hot = hots[0];

  const size_t bhq = (size_t)b * a.Hq + h, bhk = (size_t)b * a.Hkv + kh;
  v8i qf[QB][KS], df[QB][VS];
  // scale bytes: those of k-steps 2 i and 2 i + 1 in bytes 0 and 2 of word i
  // (KW, VW words of a row's D / 32 bytes, read as one dword each where the
  // bytes come in fours, and shifted to the lane half's)
  constexpr int KW = (KS + 1) / 2, VW = (VS + 1) / 2;
  int qsc[QB][KW], dsc[QB][VW];
  auto scale_word = [&](const uint8_t* row, auto steps_tag, int i) __attribute__((always_inline)) {
    constexpr int S = decltype(steps_tag)::value;   // k-steps of the row
    if constexpr (S % 2 == 0) return (int)(*reinterpret_cast<const uint32_t*>(row + 4 * i) >> (8 * hf));
    else if (2 * i + 1 < S) return (int)(row[4 * i + hf] | (uint32_t)row[4 * i + 2 + hf] << 16);
    else return (int)row[4 * i + hf];
  };
  constexpr std::integral_constant<int, KS> KTAG{};
  constexpr std::integral_constant<int, VS> VTAG{};
  // B operand of the score's rank-2 update: isolated-channel value (lanes
  // < 32), -LSE / tau (lanes >= 32) of the lane's query
  float qv[QB];
  float qv12[QB] = {};   // NH = 3: channel 1 (lanes < 32) and 2 (lanes >= 32) of the lane's query
#pragma unroll
  for (int u = 0; u < QB; u++) {
    const int qi = q0 + 32 * u + li;
    const size_t row = bhq * N + (q0 + 32 * u < L.q ? qi : 0);
#pragma unroll
    for (int s = 0; s < KS; s++) {
      qf[u][s] = frag_rows_global(a.q_code + row * DQK, s, hf);
#pragma unroll
      for (int i = 0; i < NH; i++) clear_channel(qf[u][s], s, hf, hots[i]);
    }
#pragma unroll
    for (int i = 0; i < KW; i++) qsc[u][i] = scale_word(a.q_scale + row * (DQK / 32), KTAG, i);
#pragma unroll
    for (int s = 0; s < VS; s++) df[u][s] = frag_rows_global(a.do_code + row * DV, s, hf);
#pragma unroll
    for (int i = 0; i < VW; i++) dsc[u][i] = scale_word(a.do_scale + row * (DV / 32), VTAG, i);
    const float qhot = hot >= 0 ? row_value<DQK>(a.q_code, a.q_scale, (int64_t)row, hot) : 0.f;
    qv[u] = hf ? neg_lse_over_tau(a.lse[row], a.tau) : qhot;
    if constexpr (NH == 3) {
      if (hot >= 0) qv12[u] = row_value<DQK>(a.q_code, a.q_scale, (int64_t)row, hf ? hots[2] : hots[1]);
    }
  }
  // each row's sums over the groups: of P dP in lanes < 32, of P in lanes >= 32
  double sum[QB] = {};

  const uint8_t* kcode = a.k_code + bhk * Nk * DQK;
  const uint8_t* kscale = a.k_scale + bhk * Nk * (DQK / 32);
  const uint8_t* vcode = a.v_code + bhk * Nk * DV;
  const uint8_t* vscale = a.v_scale + bhk * Nk * (DV / 32);
  // key tiles up to the block's last query, or over all keys; the first
  // nfull hold only keys that every query of the workgroup sees
  const int kend = causal ? ((qb + 1) * BQ < L.q ? (qb + 1) * BQ : L.q) : L.k;
  const int ntiles = (kend + BK - 1) / BK;
  const int nfull = causal ? qb * (BQ / BK) : L.k / BK;

  // loads of tile j0 (raw isolated-channel bytes in registers, decoded when
  // they are stored to LDS)
  uint32_t khc[NH] = {}, khs[NH] = {};
  RowLoads<DQK, NW, BK> kload;
  RowLoads<DV, NW, BK> vload;
  kload.init(w, lane);
  vload.init(w, lane);
  auto issue = [&](lds8* st, int j0) __attribute__((always_inline)) {
    // keys past the sequence read as zero (never the padding)
    kload.issue(st + C::K_OFF, kcode, j0, L.k, w);
    vload.issue(st + C::V_OFF, vcode, j0, L.k, w);
    dma_row_scales<DQK, NW, BK>(st + C::KS_OFF, kscale, j0, L.k, w, lane, 0);
    dma_row_scales<DV, NW, BK>(st + C::VS_OFF, vscale, j0, L.k, w, lane, 1);
    if (hot >= 0 && threadIdx.x < BK) {
      const int r = j0 + (int)threadIdx.x < L.k ? j0 + (int)threadIdx.x : L.k - 1;
#pragma unroll
      for (int i = 0; i < NH; i++) {
        khc[i] = kcode[(int64_t)r * DQK + hots[i]];
        khs[i] = kscale[(int64_t)r * (DQK / 32) + hots[i] / 32];
      }
    }
    __builtin_amdgcn_sched_barrier(0);   // keep every load ahead of the tile's compute
  };
  auto finish = [&](uint8_t* st) __attribute__((always_inline)) {
    if (threadIdx.x < BK) {
      float* kh = reinterpret_cast<float*>(st + C::KH_OFF) + threadIdx.x;
      kh[0] = hot >= 0 ? scaled_value(khc[0], khs[0]) : 0.f;
      kh[BK] = 1.0f;
      if constexpr (NH == 3) {
        kh[2 * BK] = hot >= 0 ? scaled_value(khc[1], khs[1]) : 0.f;
        kh[3 * BK] = hot >= 0 ? scaled_value(khc[2], khs[2]) : 0.f;
      }
    }
  };

  // A operands of one group: K and V fragments with their scale bytes, the
  // rank-2 operands
  v8i kf[KS], vf[VS];
  int ks[KW], vs[VW];
  float ka = 0.f, ka12 = 0.f;
  auto read_k = [&](const uint8_t* st, int g, int t) __attribute__((always_inline)) {
    kf[t] = frag_rows_swz<DQK>(st + C::K_OFF + 32 * g * DQK, li, t, hf);
    if (t % 2 == 1 || t == KS - 1) ks[t / 2] = scale_word(st + C::KS_OFF + 32 * g * (DQK / 32) + li * (DQK / 32), KTAG, t / 2);
  };
  auto read_v = [&](const uint8_t* st, int g, int t) __attribute__((always_inline)) {
    vf[t] = frag_rows_swz<DV>(st + C::V_OFF + 32 * g * DV, li, t, hf);
    if (t % 2 == 1 || t == VS - 1) vs[t / 2] = scale_word(st + C::VS_OFF + 32 * g * (DV / 32) + li * (DV / 32), VTAG, t / 2);
  };
  auto read_a = [&](const uint8_t* st, int g) __attribute__((always_inline)) {
    const float* kh = reinterpret_cast<const float*>(st + C::KH_OFF) + 32 * g + ((hf ? BK : 0) + li);
    ka = kh[0];
    if constexpr (NH == 3) ka12 = kh[2 * BK];
  };
  auto read_group = [&](const uint8_t* st, int g) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < KS; t++) read_k(st, g, t);
    read_a(st, g);
#pragma unroll
    for (int t = 0; t < VS; t++) read_v(st, g, t);
  };

  // The unit's MFMAs in order: S over the channels, its rank-2 update (S + k_c* q_c* - LSE / tau), dP
  constexpr int NM = KS + 1 + VS;
  auto mfma_step = [&](int m, int u, v16f& s, v16f& dp) __attribute__((always_inline)) {
    if (m < KS) {
      const v16f c = m == 0 ? v16f{} : s;
      if (m % 2 == 0) s = mfma_mx_sel<0, 0>(kf[m], qf[u][m], c, ks[m / 2], qsc[u][m / 2]);
      else s = mfma_mx_sel<2, 2>(kf[m], qf[u][m], c, ks[m / 2], qsc[u][m / 2]);
    } else if (m == KS) {
      s = rank2_update(ka, qv[u], s);
      if constexpr (NH == 3) s = rank2_update(ka12, qv12[u], s);
    } else {
      const int t = m - KS - 1;
      const v16f c = t == 0 ? v16f{} : dp;
      if (t % 2 == 0) dp = mfma_mx_sel<0, 0>(vf[t], df[u][t], c, vs[t / 2], dsc[u][t / 2]);
      else dp = mfma_mx_sel<2, 2>(vf[t], df[u][t], c, vs[t / 2], dsc[u][t / 2]);
    }
  };
  auto reread_step = [&](int m, const uint8_t* st, int g) __attribute__((always_inline)) {
    if (m < KS) read_k(st, g, m);
    else if (m == KS) read_a(st, g);
    else read_v(st, g, m - KS - 1);
  };

  // Vector work of a unit: P (mask: the group holding the wave's diagonal,
  // keys after the query), then the group's sums of P dP and P.  The lane
  // holds keys 8 (r/4) + 4 hf + r % 4 of the group, one query, and sums them
  // in this order (FP32, COMP: FP64); one exchange then gives lanes < 32 both
  // halves' sums of P dP, lanes >= 32 those of P, whose total each adds to
  // its FP64 sum.
  float p[16];
  float pn, pd;
  double qn, qd;
  auto elem_p = [&](int r, const v16f& s, bool diag) __attribute__((always_inline)) {
    p[r] = bwd_prob(s[r], a.c);
    if (diag) p[r] = (8 * (r >> 2) + 4 * hf + (r & 3)) > li ? 0.f : p[r];
    if constexpr (COMP) qd = r == 0 ? (double)p[r] : qd + (double)p[r];
    else pd = r == 0 ? p[r] : pd + p[r];
  };
  auto elem_n = [&](int r, const v16f& dp) __attribute__((always_inline)) {
    if constexpr (COMP) qn = r == 0 ? (double)p[r] * (double)dp[r] : __builtin_fma((double)p[r], (double)dp[r], qn);   // exact products
    else pn = r == 0 ? p[r] * dp[r] : __builtin_fmaf(p[r], dp[r], pn);
  };
  auto add_sums = [&](int u) __attribute__((always_inline)) {
    if constexpr (COMP) {
      const uint64_t a = __builtin_bit_cast(uint64_t, qn), b = __builtin_bit_cast(uint64_t, qd);
      const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)a, (uint32_t)b, false, false);
      const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
      sum[u] += __builtin_bit_cast(double, (uint64_t)lo[0] | (uint64_t)hi[0] << 32) +
                __builtin_bit_cast(double, (uint64_t)lo[1] | (uint64_t)hi[1] << 32);
    } else {
      const Pair t = permlane32_swap(pn, pd);
      sum[u] += (double)(t.lo + t.hi);
    }
    asm volatile("" : "+v"(sum[u]));   // here, not after later units
  };
  // items 0 .. 19 of the vector work, in order: P of element i, product of
  // element i - 4 (so that the last MFMA has finished before dP is read)
  constexpr int LAG = 4, NI = 16 + LAG;
  auto item = [&](int i, const v16f& s, const v16f& dp) __attribute__((always_inline)) {
    if (i < 16) elem_p(i, s, false);
    if (i >= LAG) elem_n(i - LAG, dp);
  };

  auto pin = [&]() __attribute__((always_inline)) {
    if constexpr (COMP) asm volatile("" : "+v"(qn), "+v"(qd));
    else asm volatile("" : "+v"(pn), "+v"(pd));
  };

  v16f s0, dp0, s1, dp1;
  // MFMAs of block uo of the group in registers into (so, dpo), interleaved
  // with the vector work of (si, dpi), the unit before it (block ui); with
  // reread, the operands of group g of st replace each one as it is used
  auto phase = [&](int uo, v16f& so, v16f& dpo, int ui, const v16f& si, const v16f& dpi, bool reread,
                   const uint8_t* st, int g) __attribute__((always_inline)) {
#pragma unroll
    for (int m = 0; m < NM; m++) {
      mfma_step(m, uo, so, dpo);
      __builtin_amdgcn_sched_barrier(0);
      if (reread) reread_step(m, st, g);
#pragma unroll
      for (int i = m * NI / NM; i < (m + 1) * NI / NM; i++) item(i, si, dpi);
      if (m == NM - 1) add_sums(ui);
      else pin();
      if (m <= KS) asm volatile("" : "+v"(so));
      else asm volatile("" : "+v"(dpo));
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto drain = [&](int ui, const v16f& si, const v16f& dpi) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NI; i++) item(i, si, dpi);
    add_sums(ui);
  };

  // Tiles t, in buffers alternating with t: the loads of tile t + 1 are in
  // flight during tile t; before tile t's last unit a barrier ends the reads
  // of its buffer, and the loads of tile t + 2 go there.
  auto turn = [&](uint8_t* cur, uint8_t* nxt, int t) __attribute__((always_inline)) {
    if (t + 1 < ntiles) finish(nxt);
    lds_barrier();
    if (t + 2 < ntiles) issue((lds8*)cur, (t + 2) * BK);
  };
  // One full tile: on entry its first group is in registers and, except at
  // the first tile (first), the unit before it is in s1 / dp1.
  auto tile_full = [&](uint8_t* cur, uint8_t* nxt, int t, bool first) __attribute__((always_inline)) {
#pragma unroll
    for (int g = 0; g < NG; g++) {
      const bool last = g == NG - 1;
      const uint8_t* src = last ? nxt : cur;
      const int gn = last ? 0 : g + 1;
      if constexpr (QB == 2) {
        // at the first unit of all there is no vector work yet: its items run on zeros (P = 1 of zero scores, dP zero) and are dropped
        phase(0, s0, dp0, 1, s1, dp1, false, src, gn);
        if (first && g == 0) sum[1] = 0.0;
        if (last) turn(cur, nxt, t);
        phase(1, s1, dp1, 0, s0, dp0, true, src, gn);
      } else {
        if (last) turn(cur, nxt, t);
        if (g & 1) {
          phase(0, s1, dp1, 0, s0, dp0, true, src, gn);
        } else {
          phase(0, s0, dp0, 0, s1, dp1, true, src, gn);
          if (first && g == 0) sum[0] = 0.0;
        }
      }
    }
  };
  // A tile of which the wave may see only some groups, one unit at a time.
  auto tile_edge = [&](const uint8_t* st, int j0) __attribute__((always_inline)) {
    for (int g = 0; g < NG; g++) {
      const int g0 = j0 + 32 * g;              // first key of the group
      if (!live || g0 >= (causal ? q0 + 32 * QB : L.k)) break;
      read_group(st, g);
#pragma unroll
      for (int u = 0; u < QB; u++) {
        const int qu = q0 + 32 * u;
        if (causal && g0 > qu) continue;       // in the block's future
#pragma unroll
        for (int m = 0; m < NM; m++) mfma_step(m, u, s0, dp0);
        const bool diag = causal && g0 == qu;
#pragma unroll
        for (int r = 0; r < 16; r++) elem_p(r, s0, diag);
#pragma unroll
        for (int r = 0; r < 16; r++) elem_n(r, dp0);
        add_sums(u);
      }
    }
  };

  issue((lds8*)stA, 0);
  finish(stA);
  lds_barrier();
  if (ntiles > 1) issue((lds8*)stB, BK);
  if (nfull > 0) {
    read_group(stA, 0);
#pragma unroll
    for (int r = 0; r < 16; r++) { s1[r] = 0.f; dp1[r] = 0.f; }
    tile_full(stA, stB, 0, true);
    for (int t = 1; t < nfull; t += 2) {
      tile_full(stB, stA, t, false);
      if (t + 1 >= nfull) break;
      tile_full(stA, stB, t + 1, false);
    }
    drain(QB - 1, s1, dp1);
  }
  for (int t = nfull; t < ntiles; t++) {
    uint8_t* cur = t & 1 ? stB : stA;
    tile_edge(cur, t * BK);
    turn(cur, t & 1 ? stA : stB, t);
  }
#pragma unroll
  for (int u = 0; u < QB; u++) {
    const int qi = q0 + 32 * u + li;
    const double n = sum[u], m = __shfl_xor(sum[u], 32);   // in lanes < 32
    if (q0 + 32 * u >= L.q || hf != 0) continue;
    const double d = m > 0.0 ? n / m : 0.0;
    const float hi = (float)d;
    const float lo = (float)(d - (double)hi);
    *reinterpret_cast<float2*>(a.delta_out + (bhq * N + qi) * 2) = make_float2(hi, lo);
  }
}

template <int DQK, int DV, int QB>
static hipError_t delta_launch(const AttnArgs& a, hipStream_t s) {
  using C = DeltaCfg<DQK, DV, 1, QB>;
  const int64_t nqb = (a.N + C::BQ - 1) / C::BQ;
  const dim3 grid((unsigned)(nqb * a.Hq * a.B));
  if (a.iso3) {
    if (a.causal) hipLaunchKernelGGL((delta_matching_kernel<DQK, DV, true, false, 3, QB>), grid, dim3(C::NT), 0, s, a);
    else hipLaunchKernelGGL((delta_matching_kernel<DQK, DV, false, false, 3, QB>), grid, dim3(C::NT), 0, s, a);
  } else if (a.causal) {
    if (a.comp) hipLaunchKernelGGL((delta_matching_kernel<DQK, DV, true, true, 1, QB>), grid, dim3(C::NT), 0, s, a);
    else hipLaunchKernelGGL((delta_matching_kernel<DQK, DV, true, false, 1, QB>), grid, dim3(C::NT), 0, s, a);
  } else {
    if (a.comp) hipLaunchKernelGGL((delta_matching_kernel<DQK, DV, false, true, 1, QB>), grid, dim3(C::NT), 0, s, a);
    else hipLaunchKernelGGL((delta_matching_kernel<DQK, DV, false, false, 1, QB>), grid, dim3(C::NT), 0, s, a);
  }
  return hipGetLastError();
}

// Two query blocks per wave halve the LDS reads per MFMA (the kernel's second
// bound: with one block every wave reads 8 KB of fragments per 32 x 32 unit
// at d = 128, 102 of the LDS's 128 bytes a cycle at the MFMA's full rate) but
// double the smallest piece of work, so they pay once the launch still fills
// the chip about twice: measured with one / two blocks at d = 128, 16 or 64
// heads, causal: 1024 workgroups of two 171 / 159 us, 2048 618 / 556, 768
// 103.3 / 104.4, 512 55.1 / 56.4 and 180 / 189 (twice the rows), 256 60 / 83;
// d = 64, 1024: 225 / 218; d = 256 (one workgroup per CU), 512: 331 / 268,
// 256: 94 / 122.  At 192 / 128 two blocks leave one workgroup per CU and are
// slower with the mask (217 against 203 us for 1024).
template <int DQK, int DV>
static hipError_t delta_dispatch(const AttnArgs& a, hipStream_t s) {
  if constexpr (DQK != 192) {
    using C2 = DeltaCfg<DQK, DV, 1, 2>;
    const int64_t wgs = (a.N + C2::BQ - 1) / C2::BQ * a.Hq * a.B;
    const int cus = cu_count();   // 0 if unknown
    if (cus > 0 && wgs >= (int64_t)2 * cus * C2::WGS) return delta_launch<DQK, DV, 2>(a, s);
  }
  return delta_launch<DQK, DV, 1>(a, s);
}

hipError_t launch_delta_matching(const AttnArgs& a, int dqk, int dv, hipStream_t s) {
  if (dqk == 64 && dv == 64) return delta_dispatch<64, 64>(a, s);
  if (dqk == 128 && dv == 128) return delta_dispatch<128, 128>(a, s);
  if (dqk == 256 && dv == 256) return delta_dispatch<256, 256>(a, s);
  if (dqk == 192 && dv == 128) return delta_dispatch<192, 128>(a, s);
  return hipErrorInvalidValue;
}

}  // namespace afp8
