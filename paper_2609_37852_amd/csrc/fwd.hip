// Forward pass (Sec. 2.3; App. B.6.2 with power-of-two probability scales).
//
// Workgroup: NW waves, 32 queries each, one (batch, query head).  Key tiles of
// BK = 128 keys (64 at 192 / 128 heads; K row codes [BK][Dqk], V col codes
// [Dv][BK], their scales) reach LDS by direct loads, double-buffered: later
// tiles stream in while the current one is computed, one barrier per tile.
// Tiles run from key 0 up to the causal diagonal (to the last key without the
// mask), so the workgroups of one KV head that run together read the same
// tiles.
//
// Per wave, in 64-key units of two aligned 32-key groups:
//   S^T = K Q^T       MX MFMA, A = K row tile (LDS), B = Q row codes (regs);
//                     lane l owns query l % 32 and holds 16 keys of each
//                     group, so row reductions are in-lane plus one exchange
//                     with lane l ^ 32.  The isolated score channel (if any)
//                     is cleared in Q and its exact product added by one
//                     FP32 rank-1 MFMA update.
//   M = integer running reference for x = S tau log2e (ceil of the row max,
//       raised lazily).  When it is raised, O and l are multiplied by
//       2^(M_old - M_new), an exact power of two (decided per wave).
//   p = 2^(x - M) (FP32, before any cast) feeds l.
//   group g: E_g = smallest integer with 2^(x_g - M) <= 448 * 2^E_g (x_g the
//       group max), codes C8(p / 2^E_g) -- the group's probability scale.
//       Since M is an integer the codes equal C8(2^(x - E)) with E the
//       group's absolute exponent, whatever the running max was.
//   O^T += V^T P^T    MX MFMA, A = V col tile (LDS), B = probability codes
//                     from registers, put in natural key order by one
//                     v_permlane32_swap per dword pair.
// Units that hold keys some query does not see (the last tiles) take a masked
// body of their own; units wholly in a wave's future are skipped.
// Epilogue: O = O_acc / l (bf16 or fp32), LSE = (M + log2 l) ln 2.
#include <type_traits>

#include "common.hpp"
#include "dma.hpp"
#include "kernels.hpp"
#include "tiles.hpp"

namespace afp8 {

constexpr float kLog2_448 = 8.807354922057604f;
// The reference M is raised only once some row's maximum exceeds it by more
// than this many powers of two: until then p = 2^(x - M) <= 2^16 simply
// accumulates larger, which FP32 holds exactly in range.  Rescales are exact
// powers of two and the codes do not depend on M, so O and l come out the
// same whenever the rescales happen.
constexpr float kLazyRescale = 16.0f;

// NH: isolated score channels (1, or 3 with ATTN_FP8_FLAG_ISOLATE3)
template <int DQK, int DV, int NH = 1>
struct FwdCfg {
  static constexpr int NW = 4, NT = 64 * NW, BQ = 32 * NW;
  static constexpr int al16(int x) { return (x + 15) & ~15; }
  // Workgroups per CU: two (two waves a SIMD) where 256 VGPRs hold a wave; at
  // dv = 256 its O accumulators alone take 128, so there it is one.
  static constexpr int WGS = DV > 128 ? 1 : 2;
  static constexpr int k_bytes(int bk) { return al16(bk * DQK + bk * DQK / 32) + bk * 4 * NH; }
  static constexpr int v_bytes(int bk) { return DV * bk + DV * 4; }
  // 128-key tiles where two buffers of each fit, else 64-key tiles (192 /
  // 128 heads).  A tile's V is read one 64-key unit later than its K, so with
  // one unit per tile V takes a third buffer.
  static constexpr int BK = 2 * (k_bytes(128) + v_bytes(128)) * WGS <= 158 * 1024 ? 128 : 64;
  // MFMAs that an LDS operand is read ahead of its own.  With dv = 128 two
  // spill: 0.744 against 0.734 ms at d = 128; at 192 / 128 242 against 238 us
  // where two workgroups share a compute unit, 46.5 against 47.4 where one has it
  // to itself, and with three isolated channels 357 against 292 us.
  static constexpr int AHEAD = DV == 128 ? 1 : 2;
  static constexpr int U = BK / 64, NVB = U == 1 ? 3 : 2;
  // K part: row codes [BK][DQK], swizzled; row scales [BK][DQK/32]; isolated-channel key values [NH][BK] FP32
  static constexpr int KS_OFF = BK * DQK, KH_OFF = al16(KS_OFF + BK * DQK / 32), KST = KH_OFF + BK * 4 * NH;
  // V part: col codes [DV][BK], swizzled; col scales [DV][4] (BK/32 used)
  static constexpr int VS_OFF = DV * BK, VST = VS_OFF + DV * 4;
  static_assert(KST == k_bytes(BK) && VST == v_bytes(BK), "stage layout");
  static_assert(DV <= NT, "one V scale word per thread");
  static_assert(BQ % BK == 0, "a query block's diagonal starts a key tile");
  static_assert(WGS * (2 * KST + NVB * VST) <= 158 * 1024, "LDS of the forward");
};

// A wave's work is a sequence of 64-key units (two aligned 32-key groups).
// One phase runs, interleaved one MFMA at a time, the scores of unit i + 1,
// the P V product of unit i - 1 and the vector work of unit i between them: a
// wave issues in order, so vector work placed after a run of MFMAs would wait
// until the last of them has issued, 64 cycles each.  Each MFMA's operands
// are read from LDS one or two MFMAs ahead.  Bound: vector issue (busy 66 % of
// the cycles: 4 of 4.6 instructions a pair are the method's own, half a
// three-way max, the exponential and its fma, the sum, half a cast, of which
// the exponential and the cast take two slots), the MFMA pipe 41 %, one or the
// other 86 %.  On 4 x 8192 tokens, 16 / 4 heads, causal, d = 128: 0.838 ms with
// one unit's products and vector work after another, 0.732 so (d = 64 0.346 ->
// 0.284 with 2 x 16 heads, d = 256 0.486 -> 0.369, 192 / 128 0.277 -> 0.249).
//
// Tiles: before the phase of tile t's last unit a barrier makes K of tile
// t + 1 and V of tile t visible, and the loads of K of tile t + 2 and V of
// tile t + 1 are issued into the buffers that no later phase reads.

// CAUSAL: the mask (key length = query length) or every key of Nk; a
// template parameter, so the causal kernel carries no key-length arithmetic.
// NH: isolated score channels; with 3, the first two share one rank-2 FP32
// MFMA (its two k slots) and the third takes a second one.
template <int DQK, int DV, bool CAUSAL, int NH = 1>
__global__ __launch_bounds__(256, (FwdCfg<DQK, DV, NH>::WGS)) void fwd_kernel(AttnArgs a) {
  using C = FwdCfg<DQK, DV, NH>;
  constexpr int NW = C::NW, BQ = C::BQ, BK = C::BK, U = C::U;
  constexpr int KS = DQK / 64, CB = DV / 32;
  // every buffer is its own object, so the compiler can tell loads into one
  // from reads of another
  __shared__ __attribute__((aligned(16))) uint8_t kA[C::KST];
  __shared__ __attribute__((aligned(16))) uint8_t kB[C::KST];
  __shared__ __attribute__((aligned(16))) uint8_t vA[C::VST];
  __shared__ __attribute__((aligned(16))) uint8_t vB[C::VST];
  __shared__ __attribute__((aligned(16))) uint8_t vC[C::NVB == 3 ? C::VST : 16];
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
  const int q0 = qb * BQ + 32 * w;
  const bool live = q0 < L.q;
  const int qi = q0 + li;
  // keys j0 .. visible to the wave's queries start groups before klim (a
  // multiple of 32): the diagonal group's end when causal, else the key length
  const int klim = causal ? q0 + 32 : L.k;
  int hots[NH];
  if constexpr (NH == 1) hots[0] = select_hot_channel<DQK>(a.q_amax, a.k_amax, b, kh, a.Hq, a.Hkv, a.G, hot_slot);
  else select_hot_channels<DQK, NH>(a.q_amax, a.k_amax, b, kh, a.Hq, a.Hkv, a.G, hot_slot, hots);
  const int hot = hots[0];

  const size_t bhq = (size_t)b * a.Hq + h, bhk = (size_t)b * a.Hkv + kh;
  const uint8_t* kcode = a.k_code + bhk * Nk * DQK;
  const uint8_t* kscale = a.k_scale + bhk * Nk * (DQK / 32);
  const uint8_t* vcode = a.vc_code + bhk * DV * Nk;
  const uint8_t* vscale = a.vc_scale + bhk * DV * (Nk / 32);

  v8i qf[KS];
  int qsc[KS];
  float qv = 0.f;     // B operand of the isolated channel's rank-1 update (lanes < 32)
  float qv2 = 0.f;    // NH = 3: qv holds channel 0 (lanes < 32) and 1 (lanes >= 32), qv2 channel 2
  {
    const size_t row = bhq * N + (live ? qi : 0);
#pragma unroll
    for (int s = 0; s < KS; s++) {
      qf[s] = frag_rows_global(a.q_code + row * DQK, s, hf);
      qsc[s] = a.q_scale[row * (DQK / 32) + 2 * s + hf];
#pragma unroll
      for (int i = 0; i < NH; i++) clear_channel(qf[s], s, hf, hots[i]);
    }
    if constexpr (NH == 1) {
      if (hot >= 0 && hf == 0) qv = row_value<DQK>(a.q_code, a.q_scale, (int64_t)row, hot);
    } else if (hot >= 0) {
      qv = row_value<DQK>(a.q_code, a.q_scale, (int64_t)row, hf ? hots[1] : hots[0]);
      if (hf == 0) qv2 = row_value<DQK>(a.q_code, a.q_scale, (int64_t)row, hots[2]);
    }
  }

  v16f oacc[CB];
#pragma unroll
  for (int cb = 0; cb < CB; cb++)
#pragma unroll
    for (int r = 0; r < 16; r++) oacc[cb][r] = 0.f;
  float M = -__builtin_inff();
  float lsum = 0.f;                           // the lane's keys' exponentials, keys ascending
  const float c = a.c;
  // key tiles up to the block's diagonal, or over all keys; the first nfull
  // hold only keys that every query of the workgroup sees
  const int ktiles = (L.k + BK - 1) / BK;
  const int ntiles = causal && (qb + 1) * (BQ / BK) < ktiles ? (qb + 1) * (BQ / BK) : ktiles;
  const int nfull = causal ? qb * (BQ / BK) : L.k / BK;

  // Loads of a tile: codes and K scales straight to LDS; the V col scales
  // (BK / 32 strided bytes per channel) and the isolated-channel bytes of
  // each key through registers, written by finish_k() / finish_v().  With
  // three isolated channels and 64-key tiles thread 64 n + key takes channel n
  // of that key (SPREAD); the first BK threads take all of theirs elsewhere.
  // SPREAD saves four registers a lane where they spill (192 / 128, 2 x 4096
  // tokens, causal: 258 against 292 us); 128-key tiles are up to 3 % slower so.
  constexpr bool SPREAD = NH == 3 && U == 1;
  constexpr int KH = SPREAD ? 1 : NH;
  uint32_t vsr[BK / 32] = {};
  uint32_t khc[KH] = {}, khs[KH] = {};
  RowLoads<DQK, NW, BK> kload;
  ColLoads<DV, NW, BK> vload;
  kload.init(w, lane);
  vload.init(w, lane, Nk);
  // keys past the sequence: K rows read as zero, V cols as its last ones (never the padding)
  auto issue_k = [&](lds8* st, int j0) __attribute__((always_inline)) {
    kload.issue(st, kcode, j0, L.k, w);
    dma_row_scales<DQK, NW, BK>(st + C::KS_OFF, kscale, j0, L.k, w, lane, 0);
    if constexpr (SPREAD) {
      if (hot >= 0 && w < NH) {
        const int r = j0 + lane < L.k ? j0 + lane : L.k - 1, ch = w == 0 ? hots[0] : w == 1 ? hots[1] : hots[NH - 1];
        khc[0] = kcode[(int64_t)r * DQK + ch];
        khs[0] = kscale[(int64_t)r * (DQK / 32) + ch / 32];
      }
    } else if (hot >= 0 && threadIdx.x < BK) {
      const int r = j0 + (int)threadIdx.x < L.k ? j0 + (int)threadIdx.x : L.k - 1;
#pragma unroll
      for (int i = 0; i < NH; i++) {
        khc[i] = kcode[(int64_t)r * DQK + hots[i]];
        khs[i] = kscale[(int64_t)r * (DQK / 32) + hots[i] / 32];
      }
    }
  };
  auto issue_v = [&](lds8* st, int j0) __attribute__((always_inline)) {
    vload.issue(st, vcode, j0, Nk, L.k, w);
    if (threadIdx.x < DV) {
#pragma unroll
      for (int g = 0; g < BK / 32; g++) {
        const int grp = (j0 + 32 * g < L.k ? j0 + 32 * g : L.k - 32) / 32;
        vsr[g] = vscale[threadIdx.x * (Nk / 32) + grp];
      }
    }
  };
  auto finish_k = [&](uint8_t* st) __attribute__((always_inline)) {
    if constexpr (SPREAD) {
      if (w < NH) reinterpret_cast<float*>(st + C::KH_OFF)[threadIdx.x] = hot >= 0 ? scaled_value(khc[0], khs[0]) : 0.f;
    } else if (threadIdx.x < BK) {
#pragma unroll
      for (int i = 0; i < NH; i++)
        reinterpret_cast<float*>(st + C::KH_OFF)[i * BK + threadIdx.x] = hot >= 0 ? scaled_value(khc[i], khs[i]) : 0.f;
    }
  };
  auto finish_v = [&](uint8_t* st) __attribute__((always_inline)) {
    if (threadIdx.x < DV) {
      if constexpr (BK == 128)
        *reinterpret_cast<uint32_t*>(st + C::VS_OFF + 4 * threadIdx.x) =
            vsr[0] | (vsr[1] << 8) | (vsr[2] << 16) | (vsr[3] << 24);
      else
        *reinterpret_cast<uint16_t*>(st + C::VS_OFF + 4 * threadIdx.x) = (uint16_t)(vsr[0] | (vsr[1] << 8));
    }
  };

  // The MFMAs of a phase.  S of a unit: the k-steps of its two groups in
  // turn (operation 2 t + g), then + k_c* q_c* of each by a rank-2 FP32 update
  // (A = isolated-channel key value, B = qv; NH = 1: qv is 0 in lanes >= 32);
  // then O of another unit, one per 32 channels.
  constexpr int NS = 2 * KS + 2, NOP = NS + CB;
  struct Opnd {
    v8i f;        // K or V fragment
    int sc;       // its scale byte
    float k0, k1; // rank-2 A operands
  };
  // operation m: K rows from Kt (64-key unit hk of the tile), V cols from Vt (unit hv)
  auto load = [&](int m, const uint8_t* Kt, int hk, const uint8_t* Vt, int hv) __attribute__((always_inline)) {
    Opnd r{};
    if (m < 2 * KS) {
      const int t = m >> 1, row0 = 64 * hk + 32 * (m & 1);
      r.f = frag_rows_swz<DQK>(Kt + row0 * DQK, li, t, hf);
      r.sc = (Kt + C::KS_OFF + row0 * (DQK / 32))[li * (DQK / 32) + 2 * t + hf];
    } else if (m < NS) {
      const float* kh0 = reinterpret_cast<const float*>(Kt + C::KH_OFF) + 64 * hk + 32 * (m - 2 * KS) + li;
      r.k0 = NH == 1 ? kh0[0] : kh0[hf ? BK : 0];
      if constexpr (NH == 3) r.k1 = hf ? 0.f : kh0[2 * BK];
    } else {
      const int ch0 = 32 * (m - NS);
      r.f = frag_rows_swz<BK>(Vt + ch0 * BK, li, hv, hf);
      r.sc = (Vt + C::VS_OFF + ch0 * 4 + 2 * hv)[li * 4 + hf];
    }
    return r;
  };
  v8i pfr = v8i{};    // B operand of the P V product: the codes of a unit's two groups
  int psc = 0;        // and the scale byte of group hf
  auto exec = [&](int m, const Opnd& r, v16f (&s)[2]) __attribute__((always_inline)) {
    if (m < 2 * KS) {
      const int t = m >> 1, g = m & 1;
      s[g] = mfma_mx(r.f, qf[t], t == 0 ? v16f{} : s[g], r.sc, qsc[t]);
      asm volatile("" : : "v"(s[g]));
    } else if (m < NS) {
      const int g = m - 2 * KS;
      s[g] = rank2_update(r.k0, qv, s[g]);
      if constexpr (NH == 3) s[g] = rank2_update(r.k1, qv2, s[g]);
      asm volatile("" : : "v"(s[g]));
    } else {
      oacc[m - NS] = mfma_mx(r.f, pfr, oacc[m - NS], r.sc, psc);
      asm volatile("" : "+v"(oacc[m - NS]));
    }
  };

  // Vector work of a unit, first part: group maxima, the reference M, the
  // group exponents.  A lane holds 16 keys (8 (r/4) + 4 hf + r % 4) of each
  // group of its query; after one exchange lanes of half g hold group g's
  // maximum, and from there work on that group alone.  O is rescaled by
  // rescale(), once the codes of the unit before are in it: their scale byte
  // cannot take a factor below its range.
  float nM;           // -M
  float sc2[2];       // 2^E of the two groups
  int ne;             // scale byte of group hf (for the P V product of this unit)
  bool raised;        // M was raised: by which factor O shrinks
  float alpha;
  auto maxima = [&](const v16f (&s)[2]) __attribute__((always_inline)) {
    float gm[2];
#pragma unroll
    for (int g = 0; g < 2; g++) {
      gm[g] = -__builtin_inff();
#pragma unroll
      for (int r = 0; r < 16; r++) gm[g] = __builtin_fmaxf(gm[g], s[g][r]);
    }
    const Pair pm = permlane32_swap(gm[0], gm[1]);
    const float own = __builtin_fmaxf(pm.lo, pm.hi);     // raw score units
    // M is raised where some row's maximum exceeds it by 2^kLazyRescale (from
    // -inf at the first unit)
    raised = __any(own * c > M + kLazyRescale);
    if (raised) {
      const float mnew = __builtin_fmaxf(M, __builtin_ceilf(__builtin_fmaxf(own, partner(own)) * c));
      const float df = __builtin_fmaxf(M - mnew, -300.f);  // M is -inf at first
      const int d = (int)df;                              // 0 for lanes whose maximum did not move
      alpha = d < -126 ? 0.f : exp2i(d);
      lsum *= alpha;
      M = mnew;
    }
    nM = -M;
    // smallest E with 2^(x_g - M) <= 448 * 2^E, kept in the normal FP32 range
    const int e0 = (int)__builtin_ceilf(__builtin_fmaf(own, c, nM) - kLog2_448);
    const int e = e0 < -126 ? -126 : e0;
    ne = e + 127;
    const auto ee = __builtin_amdgcn_permlane32_swap((uint32_t)e, (uint32_t)e, false, false);
    sc2[0] = exp2i((int)ee[0]);
    sc2[1] = exp2i((int)ee[1]);
  };
  auto rescale = [&]() __attribute__((always_inline)) {
    if (!raised) return;
#pragma unroll
    for (int cb = 0; cb < CB; cb++)
#pragma unroll
      for (int r = 0; r < 16; r++) oacc[cb][r] *= alpha;
  };
  // Second part, in pairs of elements (pair j: elements 2 j, 2 j + 1 of group
  // j / 8): p = 2^(x - M), its sum, the codes C8(p / 2^E), the sums and casts
  // LAG pairs after the exponentials; then the natural key order (lane half
  // hf: keys 16 hf .. 16 hf + 15 of the group).
  constexpr int LAG = 2, NITEM = 16 + LAG;
  float p[32];
  int cd[8];
  auto item = [&](int i, const v16f (&s)[2]) __attribute__((always_inline)) {
    if (i < 16) {
      const int g = i >> 3, r = 2 * (i & 7);
      p[2 * i] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[g][r], c, nM));
      p[2 * i + 1] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[g][r + 1], c, nM));
      asm volatile("" : "+v"(p[2 * i]), "+v"(p[2 * i + 1]));
    }
    const int j = i - LAG;
    if (j >= 0 && j < 16) {
      lsum += p[2 * j];
      lsum += p[2 * j + 1];
      const float sc = sc2[j >> 3];
      v2s w2 = (j & 1) ? __builtin_bit_cast(v2s, cd[j >> 1]) : __builtin_bit_cast(v2s, p[2 * j]);
      if (j & 1) w2 = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(w2, p[2 * j], p[2 * j + 1], sc, true);
      else w2 = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(w2, p[2 * j], p[2 * j + 1], sc, false);
      cd[j >> 1] = __builtin_bit_cast(int, w2);
      asm volatile("" : "+v"(lsum), "+v"(cd[j >> 1]));
    }
  };
  v8i npfr;
  auto order = [&]() __attribute__((always_inline)) {
    const v4i n0 = to_natural4(v4i{cd[0], cd[1], cd[2], cd[3]}), n1 = to_natural4(v4i{cd[4], cd[5], cd[6], cd[7]});
    npfr = v8i{n0[0], n0[1], n0[2], n0[3], n1[0], n1[1], n1[2], n1[3]};
  };

  // One phase: S of the next unit (K tile Kt, unit hk) into so, O of the unit
  // before (V tile Vt, unit hv; not in the first phase), vector work of si.
  auto phase = [&](v16f (&so)[2], const v16f (&si)[2], const uint8_t* Kt, int hk, const uint8_t* Vt, int hv,
                   auto first_tag) __attribute__((always_inline)) {
    constexpr int NO = decltype(first_tag)::value ? NS : NOP;
    constexpr int AH = C::AHEAD;
    Opnd o[AH + 1];
#pragma unroll
    for (int m = 0; m < AH; m++) o[m] = load(m, Kt, hk, Vt, hv);
    maxima(si);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = 0; m < NO; m++) {
      exec(m, o[m % (AH + 1)], so);
      __builtin_amdgcn_sched_barrier(0);
      if (m + AH < NO) o[(m + AH) % (AH + 1)] = load(m + AH, Kt, hk, Vt, hv);
#pragma unroll
      for (int i = m * NITEM / NO; i < (m + 1) * NITEM / NO; i++) item(i, si);
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (!decltype(first_tag)::value) rescale();
    order();
    pfr = npfr;
    psc = ne;
  };

  v16f s0[2], s1[2];
  auto kbuf = [&](int i) __attribute__((always_inline)) { return (i & 1) ? (uint8_t*)kB : (uint8_t*)kA; };
  auto vbuf = [&](int i) __attribute__((always_inline)) {
    const int j = i % C::NVB;
    return j == 0 ? (uint8_t*)vA : j == 1 ? (uint8_t*)vB : (uint8_t*)vC;
  };
  bool pending = false;   // loads whose register part finish_*() has still to write: K of tile pt + 1, V of tile pt
  // before the phase of the last unit of tile t (x: t modulo the buffers' period, known at compile time)
  auto turn = [&](int x, int t) __attribute__((always_inline)) {
    if (t > 0) {
      if (t + 1 < ntiles) finish_k(kbuf(x + 1));
      finish_v(vbuf(x));
    }
    lds_barrier();
    if (t + 2 < ntiles) issue_k((lds8*)kbuf(x), (t + 2) * BK);
    if (t + 1 < ntiles) issue_v((lds8*)vbuf(x + 1), (t + 1) * BK);
    pending = true;
    __builtin_amdgcn_sched_barrier(0);
  };
  constexpr std::true_type YES{};
  constexpr std::false_type NO_{};
  constexpr int PER = U == 1 ? 6 : 2;     // tiles until the buffers repeat
  // the phases of tile t: with two units, S of its second and of the next
  // tile's first; with one unit, S of the next tile's
  auto tile_full = [&](auto x_tag, int t, auto first_tag) __attribute__((always_inline)) {
    constexpr int x = decltype(x_tag)::value;
    constexpr bool F = decltype(first_tag)::value;
    if constexpr (U == 2) {
      if constexpr (F) phase(s1, s0, kbuf(x), 1, vbuf(x + C::NVB - 1), 1, YES);
      else phase(s1, s0, kbuf(x), 1, vbuf(x + C::NVB - 1), 1, NO_);
      turn(x, t);
      phase(s0, s1, kbuf(x + 1), 0, vbuf(x), 0, NO_);
    } else {
      turn(x, t);
      if constexpr (x & 1) {
        phase(s0, s1, kbuf(x + 1), 0, vbuf(x + C::NVB - 1), 0, NO_);
      } else {
        if constexpr (F) phase(s1, s0, kbuf(x + 1), 0, vbuf(x + C::NVB - 1), 0, YES);
        else phase(s1, s0, kbuf(x + 1), 0, vbuf(x + C::NVB - 1), 0, NO_);
      }
    }
  };
  // O of the unit whose codes are in pfr
  auto product = [&](const uint8_t* Vt, int hv) __attribute__((always_inline)) {
#pragma unroll
    for (int m = NS; m < NOP; m++) exec(m, load(m, Vt, 0, Vt, hv), s0);
  };
  // One unit of a tile that holds keys some query does not see: scores with
  // the unseen ones at -inf (their codes and sums are exact zeros), one after
  // the other
  auto unit_edge = [&](const uint8_t* Kt, const uint8_t* Vt, int hk, int j0) __attribute__((always_inline)) {
#pragma unroll
    for (int m = 0; m < NS; m++) exec(m, load(m, Kt, hk, Vt, hk), s0);
#pragma unroll
    for (int g = 0; g < 2; g++) {
      const int lim = (causal ? qi : L.k - 1) - (j0 + 64 * hk + 32 * g) - 4 * hf;   // last visible key, from the lane's first
#pragma unroll
      for (int r = 0; r < 16; r++) s0[g][r] = 8 * (r >> 2) + (r & 3) > lim ? -__builtin_inff() : s0[g][r];
    }
    maxima(s0);
    rescale();
#pragma unroll
    for (int i = 0; i < NITEM; i++) item(i, s0);
    order();
    pfr = npfr;
    psc = ne;
    product(Vt, hk);
  };

  issue_k((lds8*)kA, 0);
  finish_k(kA);
  if (ntiles > 1) {
    issue_k((lds8*)kB, BK);
    finish_k(kB);
  }
  issue_v((lds8*)vA, 0);
  finish_v(vA);
  lds_barrier();
  if (nfull > 0) {
#pragma unroll
    for (int m = 0; m < NS; m++) exec(m, load(m, kA, 0, vA, 0), s0);
    tile_full(std::integral_constant<int, 0>{}, 0, YES);
    int t = 1;
    while (true) {
      // PER tiles per round, from buffer position 1
      if (t >= nfull) break;
      tile_full(std::integral_constant<int, 1 % PER>{}, t++, NO_);
      if (t >= nfull) break;
      tile_full(std::integral_constant<int, 2 % PER>{}, t++, NO_);
      if constexpr (PER > 2) {
        if (t >= nfull) break;
        tile_full(std::integral_constant<int, 3 % PER>{}, t++, NO_);
        if (t >= nfull) break;
        tile_full(std::integral_constant<int, 4 % PER>{}, t++, NO_);
        if (t >= nfull) break;
        tile_full(std::integral_constant<int, 5 % PER>{}, t++, NO_);
        if (t >= nfull) break;
        tile_full(std::integral_constant<int, 0>{}, t++, NO_);
      }
    }
    product(vbuf(nfull - 1), U - 1);
  }
  for (int t = nfull; t < ntiles; t++) {
    if (pending) {
      if (t + 1 < ntiles) finish_k(kbuf(t + 1));
      finish_v(vbuf(t));
      lds_barrier();
    }
    if (live) {
      for (int hk = 0; hk < U && t * BK + 64 * hk < klim; hk++) unit_edge(kbuf(t), vbuf(t), hk, t * BK);
    }
    if (t + 1 < ntiles) {
      lds_barrier();
      if (t + 2 < ntiles) issue_k((lds8*)kbuf(t), (t + 2) * BK);
      issue_v((lds8*)vbuf(t + 1), (t + 1) * BK);
      pending = true;
    }
  }
  if (!live) return;
  const float l = lsum + partner(lsum);
  const float inv = 1.0f / l;
  // lane (query qi, half hf) holds channels 32 cb + 8 (r/4) + 4 hf + r % 4
  if (a.o_bf16) {
    uint16_t* orow = reinterpret_cast<uint16_t*>(a.o) + b * a.os[0] + (int64_t)qi * a.os[1] + h * a.os[2];
#pragma unroll
    for (int cb = 0; cb < CB; cb++)
#pragma unroll
      for (int g = 0; g < 4; g++) {
        const int ch = 32 * cb + 8 * g + 4 * hf;
        uint2 v;
        v.x = (uint32_t)f32_to_bf16(oacc[cb][4 * g] * inv) | ((uint32_t)f32_to_bf16(oacc[cb][4 * g + 1] * inv) << 16);
        v.y = (uint32_t)f32_to_bf16(oacc[cb][4 * g + 2] * inv) | ((uint32_t)f32_to_bf16(oacc[cb][4 * g + 3] * inv) << 16);
        *reinterpret_cast<uint2*>(orow + ch) = v;
      }
  } else {
    float* orow = reinterpret_cast<float*>(a.o) + b * a.os[0] + (int64_t)qi * a.os[1] + h * a.os[2];
#pragma unroll
    for (int cb = 0; cb < CB; cb++)
#pragma unroll
      for (int g = 0; g < 4; g++) {
        const int ch = 32 * cb + 8 * g + 4 * hf;
        *reinterpret_cast<float4*>(orow + ch) =
            make_float4(oacc[cb][4 * g] * inv, oacc[cb][4 * g + 1] * inv, oacc[cb][4 * g + 2] * inv,
                        oacc[cb][4 * g + 3] * inv);
      }
  }
  if (hf == 0) a.lse_out[bhq * N + qi] = (M + __builtin_amdgcn_logf(l)) * kLn2;
}

template <int DQK, int DV>
static hipError_t fwd_dispatch(const AttnArgs& a, hipStream_t s) {
  using C = FwdCfg<DQK, DV>;
  const int64_t nqb = (a.N + C::BQ - 1) / C::BQ;
  const dim3 grid((unsigned)(nqb * a.Hq * a.B));
  if (a.iso3) {
    if (a.causal) hipLaunchKernelGGL((fwd_kernel<DQK, DV, true, 3>), grid, dim3(C::NT), 0, s, a);
    else hipLaunchKernelGGL((fwd_kernel<DQK, DV, false, 3>), grid, dim3(C::NT), 0, s, a);
  } else {
    if (a.causal) hipLaunchKernelGGL((fwd_kernel<DQK, DV, true>), grid, dim3(C::NT), 0, s, a);
    else hipLaunchKernelGGL((fwd_kernel<DQK, DV, false>), grid, dim3(C::NT), 0, s, a);
  }
  return hipGetLastError();
}

hipError_t launch_fwd(const AttnArgs& a, int dqk, int dv, hipStream_t s) {
  if (dqk == 64 && dv == 64) return fwd_dispatch<64, 64>(a, s);
  if (dqk == 128 && dv == 128) return fwd_dispatch<128, 128>(a, s);
  if (dqk == 256 && dv == 256) return fwd_dispatch<256, 256>(a, s);
  if (dqk == 192 && dv == 128) return fwd_dispatch<192, 128>(a, s);
  return hipErrorInvalidValue;
}

}  // namespace afp8
