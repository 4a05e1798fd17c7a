// kia_fwd.hip -- forward of causal K-interval attention on gfx950, for fp32
// inputs (fp32 scores; three bf16 pieces per operand of P V) and bf16 inputs
// (one piece).
//
// One workgroup = RG row groups of 32 query rows of one (b, h) times KP key
// parts, one wave each. Each wave keeps its 32 Q rows in registers as the B
// operand of the canonical score sub-tile. Keys stream through LDS in chunks
// of KP 32-key tiles, one per key part, staged row-major (V in bf16 pieces, K of
// fp32 inputs as it is): K is read by rows (the score sub-tile's A operand) and
// V through transposing reads (the P V A operand). Large grids take RG = 4, KP =
// 1: 128 rows share each staged tile, so splitting V into pieces costs 44 VALU
// operations per thread and 32-key step against about 580 of a tile's weights.
// Grids too
// small to fill the chip give up row groups for key parts.
//
// Pass 1 (row extrema, App. A: amax/amin over the valid keys): score
//   sub-tiles and the raw row maximum (and minimum), merged across the two
//   lanes that share a row and, through LDS, across the key parts. bf16 scores
//   are not stored: pass 2 computes the same sub-tiles again, which costs less
//   than writing 4 bytes per pair and reading them back. fp32 scores take eight
//   times the matrix work, and most shapes keep them in U (FwdShape::KEEP).
// Pass 2 (Sec. 3 reconstruction and normalization): per key the
//   interval/level decision, kept in U for the backward (one byte, or the
//   position u), w^L and w^N from e^{b_{r+1}} (one exp2 per key), the row sums
//   W^N, W^L, and O += w V with the weight registers as the B operand (no data
//   movement). Prob-STE with Nearest also accumulates O^L = w^L V for the
//   backward. A tile that reaches a row's maximum (minimum) is swept for the
//   first index and the number of its ties. The weights are absolute once the
//   extrema are known, so the key parts' partial sums simply add (through
//   LDS); O = (sum w v) / W at the end: W >= 1 because the argmax key has
//   weight e^0 = 1, so no online rescaling. A wave whose V holds values that
//   three pieces do not (PieceCheck) takes the pass again on the fp32 MFMA.
// Exponential weight functions (softmax, BF16-exp, FP8-exp; App. A, App. D)
//   take the same two passes with the maximum only: pass 2 forms z = s - M,
//   the fp32 exponential as the weight function rounds it (kept in U) and the
//   weight, with no grid.

#include <type_traits>

#include "kia_device.hpp"
#include "kia_kernels.hpp"

namespace kia {

template <typename TI, int D, int CALIB, int RECON, bool OL, int RG, int KP>
__global__ __launch_bounds__(64 * RG * KP, (FwdShape<TI, D, RECON, OL, RG, KP>::OCC)) void fwd_kernel(FwdArgsT<TI> a) {
  using Shape = FwdShape<TI, D, RECON, OL, RG, KP>;
  constexpr int NP = Pieces<TI>::N, NC = D >= 32 ? D / 32 : 1;
  // MinMax and the resolved grid need the row minimum (resolved: for the
  // rounding margin of its far keys only)
  constexpr bool TRACKMIN = CALIB != CAL_FWM, NEAREST = RECON == REC_NEAREST;
  constexpr bool EXPW = is_exp_rec(RECON), COMPACT = compact_codes<CALIB, RECON>();
  static_assert(!EXPW || (CALIB == CAL_FWM && !OL), "exp weights use the maximum only");
  constexpr int BM = 32 * RG, CHK = 32 * KP, NT = 64 * RG * KP, NBUF = Shape::NBUF;
  // RG = 1: a wave's tile is read by no other, so it stages it itself (K, then
  // V, in one buffer of its own) and no barrier is needed
  constexpr bool PRIV = RG == 1;
  constexpr bool EX = Shape::EX;      // fp32 scores (K staged as it is)
  constexpr bool KEEP = Shape::KEEP;  // kept in U between the passes
  constexpr int SROWS = PRIV ? 32 : CHK, SNT = PRIV ? 64 : NT;
  using St = Stage<D, SROWS, SNT, TI>;
  using StK = std::conditional_t<EX, StageF32<D, SROWS, SNT>, St>;
  using Op = ScoreOp<TI, D>;
  constexpr int RS = St::RS, PS = St::PS;
  constexpr int NRED = Shape::NRED;
  // K chunks, then V chunks; at the end the key parts' sums (16-bit units; a K
  // block fits in a V block's place)
  constexpr int KSIZE = EX ? 2 * StK::SIZE : St::SIZE;
  static_assert(KSIZE <= St::SIZE, "K in V's place");
  constexpr int STG = PRIV ? KP * St::SIZE : NBUF * (KEEP ? St::SIZE : KSIZE + St::SIZE);
  constexpr int RED = Shape::RED / 2;
  constexpr int SMEM = STG > RED ? STG : RED;
  __shared__ __attribute__((aligned(16))) uint16_t smem[SMEM];
  __shared__ int Bad[EX ? RG * KP : 1];  // staged V out of range of the pieces
  __shared__ int Xc[KP > 1 ? RG * KP * 4 * 32 : 1];  // [row group][key part][field][row]

  const int tid = threadIdx.x;
  const int lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pr = wave % RG, kh = wave / RG;  // row group, key part
  const int T = a.T;
  const int nqb = (T + BM - 1) / BM;
  // heaviest (last) query blocks first; (b,h) fastest
  const int bh = blockIdx.x % a.BH;
  const int qb = nqb - 1 - (int)(blockIdx.x / a.BH);
  const int i0 = qb * BM;
  const int iw = i0 + pr * 32;
  const int row = iw + l32;
  const size_t slice = (size_t)bh * T * D;
  const TI *ks = a.k + slice, *vs = a.v + slice;
  const float Kf = (float)a.K;
  // key j is valid for this lane's row iff j <= jlim; a tile starting at js
  // holds a valid key for some row of the wave iff js <= wlim
  const int jlim = a.causal ? min(row, T - 1) : T - 1;
  const int wlim = iw >= T ? -1 : (a.causal ? min(iw + 31, T - 1) : T - 1);
  // every key j <= wmin is valid for every row of the wave
  const int wmin = a.causal ? min(iw, T - 1) : T - 1;
  const int kend = a.causal ? min(T, i0 + BM) : T;
  const int nstep = (kend + CHK - 1) / CHK;
  // this wave's tile inside a staged chunk, by rows and by columns
  const int krow = ((PRIV ? 0 : kh * 32) + l32) * StK::RS + half * (EX ? D / 2 : 8);
  const int vcol = (PRIV ? 0 : kh * 32) * RS + tr_base<D>(lane);

  Op qop;
  qop.load(a.q + slice, row < T ? row : T - 1, T, half);
  // Chunk steps: n counts the steps of both passes. A chunk is fetched into
  // registers one step ahead and stashed at the start of its own step, behind
  // which one barrier orders the stash before the reads; with two buffers the
  // reads of two steps back are ordered before the stash by the barrier in
  // between, with one by a barrier of its own.
  StK fk;
  St fv;
  auto kbuf = [&](int n) {
    return smem + (PRIV ? kh * St::SIZE : NBUF == 2 ? (n & 1) * (KEEP ? St::SIZE : KSIZE) : 0);
  };
  auto vbuf = [&](int n) {
    return PRIV || KEEP ? kbuf(n) : smem + NBUF * KSIZE + (NBUF == 2 ? n & 1 : 0) * St::SIZE;
  };
  auto stash_k = [&](int n, int t) {
    if constexpr (EX) fk.stash(reinterpret_cast<float *>(kbuf(n)), t);
    else fk.stash(kbuf(n), t);
  };
  auto scores = [&](const uint16_t *Kb) {
    if constexpr (EX) {
      Op kop;
      kop.read(reinterpret_cast<const float *>(Kb) + krow);
      return Op::tile(kop, qop);
    } else {
      const uint16_t *kr = Kb + krow;
      return score_tile<D, NP>([&](int p, int s) { return row_op(kr + p * PS + 16 * s); },
                               [&](int p, int s) { return qop.v[p][s]; });
    }
  };
  // this wave's tiles in U (the tiles of one query tile are consecutive in
  // both layouts; a wave past the last row is kept inside the field)
  float *Ut = a.st.U + ds_tile(bh, min(iw, T - 1) / 32, 0, (T + 31) / 32, a.causal) * 1024;

  // ---------------- pass 1: raw extrema --------------------------------
  float Rx = -INFINITY, Rn = INFINITY;
  const int stid = PRIV ? lane : tid, soff = PRIV ? kh * 32 : 0;
  fk.fetch(ks, soff, T, stid);
  for (int p = 0; p < nstep; ++p) {
    const int js = p * CHK + kh * 32;
    if (PRIV && js > wlim) break;
    if (!PRIV && NBUF == 1 && p > 0) lds_barrier();
    stash_k(p, stid);
    // the next chunk; after the last one pass 2's first
    const bool more = PRIV ? js + CHK <= wlim : p + 1 < nstep;
    fk.fetch(ks, (more ? (p + 1) * CHK : 0) + soff, T, stid);
    if (!PRIV) lds_barrier();
    if (js <= wlim) {
      f32x16 acc = scores(kbuf(p));
      if constexpr (KEEP) {
        float sv[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) sv[r] = acc[r];
        tile_store(Ut + (size_t)(js / 32) * 1024, lane, sv);
      }
      f32x16 lo = acc;
      if (js + 31 > wmin) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const bool valid = js + krel(r, half) <= jlim;
          if constexpr (TRACKMIN) lo[r] = valid ? acc[r] : INFINITY;
          acc[r] = valid ? acc[r] : -INFINITY;
        }
      }
#pragma unroll
      for (int r = 0; r < 16; r += 2) {
        Rx = fmaxf(fmaxf(acc[r], acc[r + 1]), Rx);
        if constexpr (TRACKMIN) Rn = fminf(fminf(lo[r], lo[r + 1]), Rn);
      }
    }
  }
  if (!PRIV || KEEP) fv.fetch(vs, soff, T, stid);
  Rx = fmaxf(Rx, __shfl_xor(Rx, 32));
  if constexpr (TRACKMIN) Rn = fminf(Rn, __shfl_xor(Rn, 32));
  if constexpr (KP > 1) {
    int *x = Xc + pr * KP * 128 + l32;
    if (half == 0) {
      x[kh * 128] = __float_as_int(Rx);
      x[kh * 128 + 32] = __float_as_int(Rn);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < KP; ++q) {
      Rx = fmaxf(Rx, __int_as_float(x[q * 128]));
      if constexpr (TRACKMIN) Rn = fminf(Rn, __int_as_float(x[q * 128 + 32]));
    }
  }
  // the extrema of the scores fl32(raw * scale) (the rounding is monotone); a
  // sum within its slack of the extreme one may round to the extremum
  const float Mx = Rx * a.scale;
  const float Mn = TRACKMIN ? Rn * a.scale : Mx;
  auto slack = [&](float x) { return fmaxf(fabsf(x) * 0x1p-22f, 0x1p-140f); };
  const float bx = fabsf(Rx) < INFINITY ? Rx - slack(Rx) : Rx;
  const float bn = fabsf(Rn) < INFINITY ? Rn + slack(Rn) : Rn;
  int ax = 0x7fffffff, an = 0x7fffffff, cx = 0, cn = 0;
  RowConst rc{};
  if constexpr (!EXPW) rc = fwd_row_const<CALIB>(Mx, Mn, a);
  const float a2 = 2.f * rc.alpha, b2 = 2.f * rc.beta, mg = rc.margin2;
  const float hic = 2.f * Kf - 0.75f;

  // ---------------- pass 2: reconstruct, normalize, O = P V ---------------
  f32x16 oacc[NC], olacc[OL ? NC : 1];
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      oacc[c][e] = 0.f;
      if constexpr (OL) olacc[c][e] = 0.f;
    }
  float WN = 0.f, WLs = 0.f;
  auto clamped = [&](float x) {
    if constexpr (CALIB == CAL_MINMAX) return __builtin_amdgcn_fmed3f(x, 0.75f, hic);
    else if constexpr (CALIB == CAL_FWM) return __builtin_amdgcn_fmed3f(x, -0.25f, hic);
    else return fminf(x, hic);
  };
  // the decisions of the wave's tile at key js from its scores: v
  auto decide = [&](int js, const f32x16 &S, float (&v)[16]) {
    const bool diag = js + 31 > wmin;  // some pair of the tile is not valid
    float *ut = Ut + (size_t)(js / 32) * 1024;
    // extrema: first index and tie count. One comparison per key and its wave
    // mask; only the few registers where a lane comes within rounding of an
    // extremum (about one key per row) are looked at.
    {
      uint64_t hit[16], any = 0;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        hit[r] = __ballot(S[r] >= bx);
        if constexpr (TRACKMIN) hit[r] |= __ballot(S[r] <= bn);
        any |= hit[r];
      }
      if (any) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          if (!hit[r]) continue;  // wave-uniform
          const int j = js + krel(r, half);
          const float s = S[r] * a.scale;
          const bool ok = j <= jlim;
          const bool ex = ok & (s == Mx);
          ax = ex ? min(ax, j) : ax;
          cx += ex ? 1 : 0;
          if constexpr (TRACKMIN) {
            const bool en = ok & (s == Mn);
            an = en ? min(an, j) : an;
            cn += en ? 1 : 0;
          }
        }
      }
    }
    // twice the position, v = 2u: a boundary (grid point or midpoint) is an
    // integer. Clamped a quarter past the outermost boundary that decides
    // (FWM: the cut 0 is one, MinMax: u = 0 is the argmin itself), so that
    // neither the extrema nor far tail keys look ambiguous. For an exponential
    // weight function v is the fp32 exponential as it rounds it (kept in U for
    // the backward; bf16-rounded already for BF16-exp).
    if constexpr (EXPW) {
      float z[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) z[r] = score_shift(S[r], a.scale, Mx);
      exp_tile<RECON>(z, v);
      if constexpr (RECON == REC_BF16EXP) {
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = bf16_rne(v[r]);
      }
      if (diag) {
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = js + krel(r, half) <= jlim ? v[r] : 0.f;
      }
      if (a.keep) tile_store(ut, lane, v);
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r) v[r] = fmaf(S[r], a2, b2);
      float f1 = 0.f, f0 = 1.f;
#pragma unroll
      for (int r = 0; r < 16; r += 2) {
        const float x = __builtin_amdgcn_fractf(clamped(v[r]));
        const float y = __builtin_amdgcn_fractf(clamped(v[r + 1]));
        f1 = fmaxf(fmaxf(x, y), f1);
        f0 = fminf(fminf(x, y), f0);
      }
      if (__any((f0 <= mg) | (1.f - f1 <= mg))) {
        // keys within rounding of a boundary (about 1e-5 of them)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float f = __builtin_amdgcn_fractf(clamped(v[r]));
          const bool amb = (f <= mg) | (1.f - f <= mg);
          if (!__any(amb)) continue;  // wave-uniform
          const float x = exact_v2<CALIB>(S[r] * a.scale, v[r], Mx, Mn, a.K, a.tau);
          v[r] = amb ? x : v[r];
        }
      }
      // the position of an extremum rounds to either side of its end of the grid:
      // t stays in [0, 1], so that a chord's weight is never below 0 or above its
      // ends (for the backward too, which reads u)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        v[r] = CALIB == CAL_MINMAX ? __builtin_amdgcn_fmed3f(v[r], 0.f, 2.f * Kf)
                                   : fminf(v[r], 2.f * Kf);
      if (diag) {
        // a position that no valid key takes and whose weight is 0: the FWM
        // tail, below the argmin (u >= 0 up to rounding), or minus infinity
        constexpr float none = CALIB == CAL_FWM ? -0.25f : CALIB == CAL_MINMAX ? -1.25f : -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = js + krel(r, half) <= jlim ? v[r] : none;
      }
      if constexpr (!COMPACT) {
        if (a.keep) {
          float u[16];
#pragma unroll
          for (int r = 0; r < 16; ++r) u[r] = 0.5f * v[r];
          tile_store(ut, lane, u);
        }
      }
    }
  };
  // its weights and their products with V (EXACT: on the fp32 MFMA, V from memory)
  auto accumulate_as = [&](int js, const float (&v)[16], const uint16_t *vb, auto tag) {
    constexpr bool EXACT = decltype(tag)::value;
    uint32_t cw[4];
    float tWN = 0.f, tWL = 0.f;  // sub-tile sums first: shorter running sums
    // the weights of the lane's keys 8 t .. 8 t + 7, the k-slots of one step
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      float w[8], wl[OL ? 8 : 1];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int r = 8 * t + e;
        if constexpr (EXPW) {
          w[e] = exp_weight_of<RECON>(v[r]);
          tWL += w[e];
        } else {
          // c = floor(2u) = 2r + [t >= 1/2], in [-1, 2K - 1] (resolved:
          // unbounded below); -1 is the FWM tail
          const float c = floorf(clamped(v[r]));
          const float hc = 0.5f * c;
          const float rf = floorf(hc);
          if constexpr (COMPACT)
            cw[r >> 2] = __builtin_amdgcn_cvt_pk_u8_f32(c + 1.f, r & 3, (r & 3) ? cw[r >> 2] : 0u);
          float arg = fmaf(rf, rc.hl, rc.b1l);
          // weight 0: the FWM tail, and keys that are not valid
          if constexpr (CALIB == CAL_FWM) arg = rf < 0.f ? -INFINITY : arg;
          if constexpr (CALIB == CAL_MINMAX) arg = v[r] < -1.f ? -INFINITY : arg;
          const float Eu = __builtin_amdgcn_exp2f(arg);
          const float El = Eu * rc.emh;
          float t01 = fmaf(v[r], 0.5f, -rf);
          if constexpr (CALIB == CAL_RESOLVED) t01 = __builtin_amdgcn_fmed3f(t01, 0.f, 1.f);
          const float wL = fmaf(t01, Eu - El, El);
          tWL += wL;
          if constexpr (NEAREST) {
            w[e] = hc > rf ? Eu : El;
            tWN += w[e];
            if constexpr (OL) wl[e] = wL;
          } else {
            w[e] = wL;
          }
        }
      }
      // (the bytes are made here: only the store below needs them, and left to
      // it they would keep the 16 positions live through the products)
      if constexpr (COMPACT) asm volatile("" : "+v"(cw[2 * t]), "+v"(cw[2 * t + 1]));
      if constexpr (EXACT) {
        const RowRead<D> rv(vs, js, T, 4 * half, l32);
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            const float x = rv.at(krel0(8 * t + e), 32 * c);
            oacc[c] = mfma32(x, w[e], oacc[c]);
            if constexpr (OL) olacc[c] = mfma32(x, wl[e], olacc[c]);
          }
        continue;
      }
      bf16x8 wo[NP], wlo[OL ? NP : 1];
      to_pieces<NP>(w, wo);
      if constexpr (OL) to_pieces<NP>(wl, wlo);
      // Two waves share a SIMD: the one in its matrix products goes first, so
      // that the other's vector work fills in behind. B8 H12 T1024 d64 fp32
      // with O_l: 179.5 -> 172 us; without O_l (half the products) and with
      // bf16 inputs it made no difference.
      if constexpr (OL && NP == 3) __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        bf16x8 av[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) av[p] = tr_op<RS>(vb + p * PS + 16 * t * RS + 32 * c);
        oacc[c] = mma<NP>(av, wo, oacc[c]);
        if constexpr (OL) olacc[c] = mma<NP>(av, wlo, olacc[c]);
      }
      if constexpr (OL && NP == 3) __builtin_amdgcn_s_setprio(0);
    }
    if constexpr (COMPACT)
      if (a.keep) codes_store(Ut + (size_t)(js / 32) * 1024, lane, cw);
    WN += tWN;
    WLs += tWL;
  };
  auto accumulate = [&](int js, const float (&v)[16], const uint16_t *vb) {
    accumulate_as(js, v, vb, std::false_type{});
  };
  PieceCheck check;  // of the V values that this thread stages
  if constexpr (KEEP) {
    // the wave's scores come back from U one tile ahead (each lane reads what
    // it wrote itself; a tile's decisions replace them after that)
    auto load_s = [&](int js, f32x16 &S) {
      float sv[16];
      tile_load(Ut + (size_t)(min(js, max(wlim, 0)) / 32) * 1024, lane, sv);
#pragma unroll
      for (int r = 0; r < 16; ++r) S[r] = sv[r];
    };
    __syncthreads();
    f32x16 S;
    load_s(kh * 32, S);
    for (int p = 0; p < nstep; ++p) {
      const int js = p * CHK + kh * 32;
      if (PRIV && js > wlim) break;
      if (!PRIV && NBUF == 1 && p > 0) lds_barrier();
      fv.stash(vbuf(p), stid, &check);
      fv.fetch(vs, min(p + 1, nstep - 1) * CHK + soff, T, stid);
      f32x16 Sn;
      load_s(js + CHK, Sn);
      if (!PRIV) lds_barrier();
      if (js <= wlim) {
        __builtin_amdgcn_sched_barrier(0);
        float v[16];
        decide(js, S, v);
        __builtin_amdgcn_sched_barrier(0);
        accumulate(js, v, vbuf(p) + vcol);
        __builtin_amdgcn_sched_barrier(0);
      }
      S = Sn;
    }
  } else if constexpr (PRIV) {
    for (int p = 0; p < nstep; ++p) {
      const int js = p * CHK + kh * 32;
      if (js > wlim) break;
      stash_k(0, lane);
      fv.fetch(vs, js, T, lane);
      __builtin_amdgcn_sched_barrier(0);
      const f32x16 S = scores(kbuf(0));
      __builtin_amdgcn_sched_barrier(0);
      // V takes K's place, the next K is fetched
      fv.stash(vbuf(0), lane, &check);
      fk.fetch(ks, min(p + 1, nstep - 1) * CHK + soff, T, lane);
      __builtin_amdgcn_sched_barrier(0);
      float v[16];
      decide(js, S, v);
      __builtin_amdgcn_sched_barrier(0);
      accumulate(js, v, vbuf(0) + vcol);
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {
    for (int p = 0; p < nstep; ++p) {
      const int js = p * CHK + kh * 32;
      if (NBUF == 1) lds_barrier();
      stash_k(nstep + p, tid);
      fv.stash(vbuf(nstep + p), tid, &check);
      const int nx = min(p + 1, nstep - 1) * CHK;
      fk.fetch(ks, nx, T, tid);
      fv.fetch(vs, nx, T, tid);
      lds_barrier();
      if (js <= wlim) {
        __builtin_amdgcn_sched_barrier(0);
        const f32x16 S = scores(kbuf(nstep + p));
        __builtin_amdgcn_sched_barrier(0);
        float v[16];
        decide(js, S, v);
        __builtin_amdgcn_sched_barrier(0);
        accumulate(js, v, vbuf(nstep + p) + vcol);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  if constexpr (EX) {
    // V out of range of the pieces: the wave's pass 2 again, scores and P V both
    // on the fp32 MFMA and their operands from memory
    bool out = __any(check.bad());
    if constexpr (!PRIV) {
      if (lane == 0) Bad[wave] = out;
      __syncthreads();
      out = any_flag<RG * KP>(Bad);
    }
    if (out) {
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          oacc[c][e] = 0.f;
          if constexpr (OL) olacc[c][e] = 0.f;
        }
      WN = 0.f, WLs = 0.f;
      ax = 0x7fffffff, an = 0x7fffffff, cx = 0, cn = 0;
      int qrow = min(row, T - 1), krow = l32, h = half;
      asm volatile("" : "+v"(qrow), "+v"(krow), "+v"(h));
#pragma unroll 1
      for (int js = kh * 32; js <= wlim; js += CHK) {
        Op ko, qo;
        qo.load(a.q + slice, qrow, T, h);
        ko.load(ks, js + krow, T, h);
        const f32x16 S = Op::tile(ko, qo);
        __builtin_amdgcn_sched_barrier(0);
        float v[16];
        decide(js, S, v);
        __builtin_amdgcn_sched_barrier(0);
        accumulate_as(js, v, nullptr, std::true_type{});
      }
    }
  }
  WN += __shfl_xor(WN, 32);
  WLs += __shfl_xor(WLs, 32);
  ax = min(ax, __shfl_xor(ax, 32));
  cx += __shfl_xor(cx, 32);
  if constexpr (TRACKMIN) {
    an = min(an, __shfl_xor(an, 32));
    cn += __shfl_xor(cn, 32);
  }
  if constexpr (KP > 1) {
    // key parts 1.. hand their partial sums to key part 0, which adds them in
    // part order (the chunk buffers are free behind the first barrier)
    __syncthreads();
    float *red = reinterpret_cast<float *>(smem) + pr * (KP - 1) * 64 * NRED + lane;
    int *xr = Xc + pr * KP * 128 + l32;
    if (kh > 0) {
      float *rk = red + (kh - 1) * 64 * NRED;
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          rk[(c * 16 + e) * 64] = oacc[c][e];
          if constexpr (OL) rk[((NC + c) * 16 + e) * 64] = olacc[c][e];
        }
      rk[(NRED - 2) * 64] = WN;
      rk[(NRED - 1) * 64] = WLs;
      if (half == 0) {
        int *x = xr + kh * 128;
        x[0] = ax; x[32] = cx; x[64] = an; x[96] = cn;
      }
    }
    __syncthreads();
    if (kh > 0) return;
#pragma unroll 1
    for (int q = 0; q < KP - 1; ++q) {
      const float *rk = red + q * 64 * NRED;
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          oacc[c][e] += rk[(c * 16 + e) * 64];
          if constexpr (OL) olacc[c][e] += rk[((NC + c) * 16 + e) * 64];
        }
      WN += rk[(NRED - 2) * 64];
      WLs += rk[(NRED - 1) * 64];
      const int *x = xr + (q + 1) * 128;
      ax = min(ax, x[0]); cx += x[32]; an = min(an, x[64]); cn += x[96];
    }
  }
  if (row >= T) return;
  const size_t ridx = (size_t)bh * T + row;
  const float W = NEAREST ? WN : WLs;
  if (half == 0) {
    a.st.M[ridx] = Mx;
    a.st.amax[ridx] = ax;
    a.st.nmax[ridx] = cx;
    if constexpr (TRACKMIN) {
      a.st.m[ridx] = Mn;
      a.st.amin[ridx] = an;
      a.st.nmin[ridx] = cn;
    }
    a.st.W[ridx] = W;
    a.st.WL[ridx] = WLs;
  }
  const float inv = 1.f / W, invl = 1.f / WLs;
  float *orow = a.o + slice + (size_t)row * D;
  uint16_t *orow16 = a.o16 + slice + (size_t)row * D;
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int n = c * 32 + 8 * g + 4 * half;
      if (n >= D) continue;
      f32x4 x = {oacc[c][4 * g] * inv, oacc[c][4 * g + 1] * inv,
                 oacc[c][4 * g + 2] * inv, oacc[c][4 * g + 3] * inv};
      if (NP == 1 && a.o16)
        *reinterpret_cast<uint2 *>(orow16 + n) =
            make_uint2(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]));
      else
        *reinterpret_cast<f32x4 *>(orow + n) = x;
      if constexpr (OL) {
        f32x4 y = {olacc[c][4 * g] * invl, olacc[c][4 * g + 1] * invl,
                   olacc[c][4 * g + 2] * invl, olacc[c][4 * g + 3] * invl};
        *reinterpret_cast<f32x4 *>(a.st.OL + ridx * D + n) = y;
      }
    }
}

#define KIA_FWD_GRID(TI, D, RG, KP)                                                         \
  template __global__ void fwd_kernel<TI, D, CAL_MINMAX, REC_LERP, false, RG, KP>(FwdArgsT<TI>);    \
  template __global__ void fwd_kernel<TI, D, CAL_MINMAX, REC_NEAREST, false, RG, KP>(FwdArgsT<TI>); \
  template __global__ void fwd_kernel<TI, D, CAL_MINMAX, REC_NEAREST, true, RG, KP>(FwdArgsT<TI>);  \
  template __global__ void fwd_kernel<TI, D, CAL_FWM, REC_LERP, false, RG, KP>(FwdArgsT<TI>);       \
  template __global__ void fwd_kernel<TI, D, CAL_FWM, REC_NEAREST, false, RG, KP>(FwdArgsT<TI>);    \
  template __global__ void fwd_kernel<TI, D, CAL_FWM, REC_NEAREST, true, RG, KP>(FwdArgsT<TI>);     \
  template __global__ void fwd_kernel<TI, D, CAL_RESOLVED, REC_LERP, false, RG, KP>(FwdArgsT<TI>);  \
  template __global__ void fwd_kernel<TI, D, CAL_RESOLVED, REC_NEAREST, false, RG, KP>(FwdArgsT<TI>); \
  template __global__ void fwd_kernel<TI, D, CAL_RESOLVED, REC_NEAREST, true, RG, KP>(FwdArgsT<TI>);
#define KIA_FWD_EXP(D, RG, KP)                                                               \
  template __global__ void fwd_kernel<float, D, CAL_FWM, REC_SOFTMAX, false, RG, KP>(FwdArgs); \
  template __global__ void fwd_kernel<float, D, CAL_FWM, REC_BF16EXP, false, RG, KP>(FwdArgs); \
  template __global__ void fwd_kernel<float, D, CAL_FWM, REC_FP8EXP, false, RG, KP>(FwdArgs);
#define KIA_FWD_F32(D, RG, KP)    \
  KIA_FWD_GRID(float, D, RG, KP)  \
  KIA_FWD_EXP(D, RG, KP)
// the launch shapes of one head dimension
#define KIA_FWD_D(D)              \
  KIA_FWD_F32(D, 4, 1)            \
  KIA_FWD_F32(D, 2, 2)            \
  KIA_FWD_F32(D, 1, 4)            \
  KIA_FWD_GRID(uint16_t, D, 4, 1) \
  KIA_FWD_GRID(uint16_t, D, 2, 2) \
  KIA_FWD_GRID(uint16_t, D, 1, 4)

// One head dimension per compilation (KIA_HEAD, set by the build).
#if KIA_HEAD == 16
KIA_FWD_D(16)
KIA_FWD_F32(16, 1, 8)
#elif KIA_HEAD == 32
KIA_FWD_D(32)
KIA_FWD_F32(32, 1, 8)
#elif KIA_HEAD == 64
KIA_FWD_D(64)
KIA_FWD_F32(64, 1, 8)
#elif KIA_HEAD == 128
KIA_FWD_D(128)
#else
#error "KIA_HEAD must name a head dimension"
#endif

}  // namespace kia
