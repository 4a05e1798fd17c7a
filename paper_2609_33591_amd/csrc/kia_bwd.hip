// kia_bwd.hip -- backward of causal K-interval attention on gfx950.
//
// Four launches on the caller's stream (App. B):
//  1. bwd_pre   per row: D^X = dO . O^X (O^X = O, or O^L for Prob-STE with
//               Nearest) and the row record (grid constants, 1/W, 1/W^X,
//               -D^X/W^X; with fp32 inputs whether dO or q leave the range of
//               the pieces, see PieceCheck); zeroes the two row sums.
//  2. bwd_main  KV-major: one workgroup per 128 keys, waves of 32 keys
//               stream 32-query tiles (staged in LDS, prefetched into
//               registers one tile ahead). The scores are not recomputed:
//               each (query, key) tile's decided positions u come from the
//               forward (stats U), so the index decisions are the forward's
//               own. dP^T on MFMA, per key (weights from u)
//               gamma = (g - D^X)/W^X, Delta, dS = gamma Delta, the row sums
//               S_self = sum dS and (MinMax) sum gamma dw^L/dM
//               (Eq. calgrad); dV += P^T dO and dK += dS^T Q through a
//               wave-private LDS transpose; dS is written to a tiled fp32
//               scratch for the dQ product.
//  3. bwd_dq    Q-major: dQ = scale (dS K + calibration terms of the row):
//               Eq. (full) puts cM = sum_j gamma_j dw_j/dM on the argmax key
//               and cm = -(S_self + cM) (from Delta + dw/dM + dw/dm = 0) on
//               the argmin key; FWM has cM = -S_self. For rows with unique
//               extrema it also scatter-adds dK_amax += scale cM q_i and
//               dK_amin += scale cm q_i. (Where the main kernel's query range is
//               in three or four parts, it first adds their dV up, see
//               BwdArgsT::fold.)
//  4. bwd_ties  (full gradient only) rows with tied extrema: recompute the
//               row's scores with the canonical sub-tile and split cM / cm
//               evenly over every key equal to M / m (edge-case table).
// The exponential weight functions (softmax, BF16-exp, FP8-exp) run the
// same launches with the FWM calibration's bookkeeping: U holds each key's
// fp32 exponential, dS = dz of the weight function, and the maximum's
// channel cM = -S_self lands on the argmax keys (z = s - M keeps M on the
// gradient path).
#include <type_traits>

#include "kia_device.hpp"
#include "kia_kernels.hpp"

namespace kia {

constexpr int BKV = 128;  // keys per bwd_main workgroup
constexpr int BQ = 32;    // queries per streamed tile

// ---------------------------------------------------------------------------
template <int D, typename TI>
__global__ __launch_bounds__(256) void bwd_pre_kernel(BwdArgsT<TI> a) {
  constexpr int L = D / 4;  // lanes per row, one float4 each
  constexpr int RPB = 256 / L;
  const int tid = threadIdx.x;
  const int sub = tid % L;
  const size_t R = (size_t)a.BH * a.T;
  const size_t ridx = (size_t)blockIdx.x * RPB + tid / L;
  const bool live = ridx < R;
  const bool probN = (a.recon == REC_NEAREST) & (a.ste == STE_PROB);
  float dot = 0.f;
  if (live && (a.dq_piece > 0 || a.fold)) {  // the dQ pieces, or parts of dV, add into dQ
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    *reinterpret_cast<f32x4 *>(a.dq + ridx * D + sub * 4) = z;
  }
  if (live && a.qsplit > 1) {  // the split main kernel adds into dK, dV
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    *reinterpret_cast<f32x4 *>(a.dk + ridx * D + sub * 4) = z;
    *reinterpret_cast<f32x4 *>(a.dv + ridx * D + sub * 4) = z;
  }
  // every load up front, from a clamped row (one memory round trip; the
  // row statistics are the same address for the row's lanes)
  const size_t rr = live ? ridx : 0;
  const float *ox = probN ? a.st.OL + rr * D : a.o + rr * D;
  // the bf16-output variant's O is bf16 (O^L stays fp32 in stats)
  const f32x4 x = (a.o16 && !probN) ? load4(a.o16 + rr * D + sub * 4)
                                    : *reinterpret_cast<const f32x4 *>(ox + sub * 4);
  const f32x4 y = load4(a.dO + rr * D + sub * 4);
  // (fp32: rows of dO or q that hold a value out of range of the pieces take the
  // main kernel's products on the fp32 MFMA)
  bool out = false;
  if constexpr (sizeof(TI) == 4) {
    const f32x4 z = load4(a.q + rr * D + sub * 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) out |= out_of_pieces(y[e]) | out_of_pieces(z[e]);
  }
  const float M = a.st.M[rr];
  const float m = a.calib != CAL_FWM && a.recon < REC_SOFTMAX ? a.st.m[rr] : M;
  const float W = a.st.W[rr];
  const float WX = probN ? a.st.WL[rr] : W;
  if (live) dot = x[0] * y[0] + x[1] * y[1] + x[2] * y[2] + x[3] * y[3];
#pragma unroll
  for (int off = L / 2; off > 0; off >>= 1) {
    dot += __shfl_xor(dot, off);
    if constexpr (sizeof(TI) == 4) out = out | (__shfl_xor(out ? 1 : 0, off) != 0);
  }
  if (live && sub == 0) {
    // the grid constants (the decision constants alpha, beta, margin are not
    // needed: the backward reads the forward's decided positions)
    RowConst rc{};  // unused by the exponential weight functions
    rc.emh = 1.f;
    if (a.recon < REC_SOFTMAX)
      grid_consts(M, m, a.K, a.calib, a.tau, rc.hl, rc.b1l, rc.emh, rc.dcoef, rc.degen);
    const float invWX = 1.f / WX;
    f32x4 *rec = reinterpret_cast<f32x4 *>(a.st.rowrec + ridx * RR_COUNT);
    const f32x4 r0 = {rc.alpha, rc.beta, rc.margin2, rc.hl};
    const f32x4 r1 = {rc.b1l, rc.emh, rc.dcoef, 1.f / W};
    const f32x4 r2 = {invWX, -dot * invWX, M, m};
    // (the sign of the flag marks a row out of range of the pieces)
    f32x4 r3 = {copysignf(rc.degen ? 1.f : 0.f, out ? -1.f : 1.f), 0.f, 0.f, 0.f};
    if (a.recon < REC_SOFTMAX) {
      const float dW = rc.dcoef * W;
      r3[1] = rc.b1l - __log2f(W);
      r3[2] = dW * invWX;
      r3[3] = -dW * dot * invWX;
    }
    rec[0] = r0; rec[1] = r1; rec[2] = r2; rec[3] = r3;
    a.st.sself[ridx] = 0.f;
    a.st.cM[ridx] = 0.f;
  }
}

// ---------------------------------------------------------------------------
// Main kernel: one workgroup = 4 waves = 128 keys of one (b, h), a wave 32 of
// them, streaming 32-query tiles of Q and dO (staged in LDS as bf16 pieces, two
// buffers, one barrier per tile; both are read by rows or through transposing
// reads as a product needs them). Per tile and wave:
//   dP^T = V dO^T with the wave's V rows in registers (lane = query, register =
//   key: the layout of the forward's decisions, and each row's constants are
//   lane-local); P and dS per key; dS to its scratch tile; then P and dS go
//   through a wave-private LDS tile as bf16 pieces, written by rows of 4 keys
//   and read back transposed, as the A operands of dV += P^T dO and
//   dK += dS^T Q.
// Three products of 24 (d = 64, fp32) MFMAs each, about 570 VALU instructions
// and 60 KiB of LDS traffic per 32x32 tile: no single unit bounds it, so two
// workgroups per CU (256 registers a wave) run out of phase; fp32 at d = 128
// needs 512.
template <typename TI, int D, int CALIB, int RECON>
__global__ __launch_bounds__(256, (MainShape<TI, D>::OCC)) void bwd_main_kernel(BwdArgsT<TI> a) {
  constexpr int NP = Pieces<TI>::N, NC = D >= 32 ? D / 32 : 1;
  using St = Stage<D, BQ, 256, TI>;
  constexpr int RS = St::RS, PS = St::PS;
  constexpr int XT = NP * 32 * 32;  // a wave's transpose tile
  __shared__ __attribute__((aligned(16))) uint16_t Tl[2][2 * St::SIZE];  // Q, dO
  __shared__ __attribute__((aligned(16))) uint16_t Xt[4 * XT];
  __shared__ float Part[2][4 * 32 * 2];

  const int tid = threadIdx.x;
  const int lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int T = a.T;
  const int nq = (T + 31) / 32;
  // key block (ascending: the longest causal key blocks first) and the part
  // of its query range (qsplit parts of nearly equal tile counts)
  const int kb = (int)(blockIdx.x / a.BH) / a.qsplit;
  const int qpart = (int)(blockIdx.x / a.BH) % a.qsplit;
  const int bh = blockIdx.x % a.BH;
  const int j0 = kb * BKV;
  const int jw = j0 + 32 * wave;
  const size_t slice = (size_t)bh * T * D;
  const TI *qs = a.q + slice, *dos = a.dO + slice;
  constexpr bool minmax = CALIB == CAL_MINMAX;
  constexpr bool nearest = RECON == REC_NEAREST;
  constexpr bool EXPW = is_exp_rec(RECON);
  constexpr bool COMPACT = compact_codes<CALIB, RECON>();
  const bool want_cm = minmax & grad_channels(a.grad);
  const float invK = 1.f / (float)a.K, Kf = (float)a.K;

  // this wave's 32 keys of V as A operands
  bf16x8 vop[NP][D / 16];
  const bool vout = __any(load_rows<D>(a.v + slice, jw + l32, T, half, vop));

  f32x16 dva[NC], dka[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int e = 0; e < 16; ++e) { dva[c][e] = 0.f; dka[c][e] = 0.f; }

  const int q0 = a.causal ? j0 : 0;
  const int ntall = (T - q0 + BQ - 1) / BQ;
  const int tb = ntall * qpart / a.qsplit, te = ntall * (qpart + 1) / a.qsplit;
  const int qstart = q0 + tb * BQ;
  const int nt = te - tb;

  // next-tile prefetch: Q and dO rows, and what the tile needs of the lane's
  // row record (a quad of it for FWM: the grid constants are the call's)
  St fq, fd;
  constexpr bool R012 = minmax && !EXPW, R12 = EXPW || R012;
  f32x4 r0, r1, r2, r3;
  auto fetch_rec = [&](int i0) {
    const int i = i0 + l32;
    const float *rr = a.st.rowrec + ((size_t)bh * T + (i < T ? i : T - 1)) * RR_COUNT;
    if constexpr (R012) r0 = *reinterpret_cast<const f32x4 *>(rr);
    if constexpr (R12) r1 = *reinterpret_cast<const f32x4 *>(rr + 4);
    if constexpr (R12) r2 = *reinterpret_cast<const f32x4 *>(rr + 8);
    if constexpr (!EXPW || NP == 3) r3 = *reinterpret_cast<const f32x4 *>(rr + 12);
  };
  // row sums of tile tp: the four waves' partials, then one atomic per row
  auto flush = [&](int tp) {
    const int ip = qstart + tp * BQ;
    if (a.grad != GRAD_DETACH && tid < 32 && ip + tid < T) {
      const float *pp = Part[tp & 1];
      float sv = 0.f, mm = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        sv += pp[(w * 32 + tid) * 2];
        mm += pp[(w * 32 + tid) * 2 + 1];
      }
      put_row_sums(a, kb, (size_t)bh * T + ip + tid, sv, mm, minmax);
    }
  };
  // transpose tile [piece][query][key]: rows of eight 4-key units, permuted by
  // the row's group of four, so that a wave's 8-byte writes and the
  // transposing reads fall in distinct banks
  uint16_t *Xw = Xt + wave * XT;
  const int xw = l32 * 32, xs = (l32 >> 2) & 7;
  const int xrow = 4 * half + ((lane & 15) >> 2), xunit = 4 * ((lane >> 4) & 1) + (lane & 3);
  auto put_tile = [&](const float (&X)[16]) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      bf16x8 w[NP];
      to_pieces<NP>(reinterpret_cast<const float(&)[8]>(X[8 * t]), w);
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        const u32x4 q = __builtin_bit_cast(u32x4, w[p]);
        uint16_t *x = Xw + p * 1024 + xw;
        *reinterpret_cast<u32x2 *>(x + 4 * ((4 * t + half) ^ xs)) = u32x2{q[0], q[1]};
        *reinterpret_cast<u32x2 *>(x + 4 * ((4 * t + 2 + half) ^ xs)) = u32x2{q[2], q[3]};
      }
    }
  };
  typedef s16x4 __attribute__((address_space(3))) *lds4;
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  // lane = key, k-slots = queries krel(8 t + e, half)
  auto get_op = [&](int t, bf16x8 (&op)[NP]) {
    const int ra = 16 * t + xrow, rb = ra + 8;
    const int oa = ra * 32 + 4 * (xunit ^ (ra >> 2)), ob = rb * 32 + 4 * (xunit ^ (rb >> 2));
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(Xw + p * 1024 + oa));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(Xw + p * 1024 + ob));
      op[p] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
  };
  // acc += X^T B with B a staged [query][d] tile and av the two k-steps of X:
  // the operands of a column block are read while the previous one's products
  // run
  auto product = [&](const bf16x8 (&av)[2][NP], const uint16_t *B, f32x16 (&acc)[NC]) {
    bf16x8 bv[2][NP];
    auto read = [&](int n) {
#pragma unroll
      for (int p = 0; p < NP; ++p)
        bv[n & 1][p] = tr_op<RS>(B + p * PS + 16 * (n / NC) * RS + 32 * (n % NC));
    };
    read(0);
#pragma unroll
    for (int n = 0; n < 2 * NC; ++n) {
      if (n + 1 < 2 * NC) read(n + 1);
      acc[n % NC] = mma<NP>(av[n / NC], bv[n & 1], acc[n % NC]);
    }
  };

  // the same on the fp32 MFMA, for operands out of range of the pieces: X (lane =
  // query, register = key) through LDS as it is, B's rows from memory
  auto product32 = [&](const float (&X)[16], const TI *B, int i0, f32x16 (&acc)[NC]) {
    typedef float f32a __attribute__((may_alias));
    f32a *x = reinterpret_cast<f32a *>(Xw);
#pragma unroll
    for (int r = 0; r < 16; ++r) x[l32 * 32 + krel(r, half)] = X[r];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const RowRead<D> rb(B, i0, T, half, l32);
#pragma unroll 1
    for (int e = 0; e < 16; ++e) {
      const float xv = x[(2 * e + half) * 32 + l32];
#pragma unroll
      for (int c = 0; c < NC; ++c) acc[c] = mfma32(xv, rb.at(2 * e, 32 * c), acc[c]);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };

  GradRange dsr;  // of the dS that went into dK by pieces
  // one 32-query tile (EXACT: its products on the fp32 MFMA)
  auto tile_as = [&](int i0, const uint16_t *Qb, const uint16_t *dOb, float &ps, float &pm,
                     auto tag) {
    constexpr bool EXACT = decltype(tag)::value;
    // the forward's decided positions of this (query, key) tile (one byte
    // per key under FWM with Nearest)
    const size_t tile = ds_tile(bh, i0 / 32, jw / 32, nq, a.causal) * 1024;
    float u[16];
    uint4 cw;
    if constexpr (COMPACT) cw = codes_load(a.st.U + tile, lane);
    else tile_load(a.st.U + tile, lane, u);
    // (nothing of the two forms is shared: it would stay live across both)
    if constexpr (EXACT && !COMPACT) {
#pragma unroll
      for (int r = 0; r < 16; ++r) asm volatile("" : "+v"(u[r]));
    }
    if constexpr (EXACT && COMPACT)
      asm volatile("" : "+v"(cw.x), "+v"(cw.y), "+v"(cw.z), "+v"(cw.w));
    const uint16_t *dr = dOb + l32 * RS + 8 * half;
    f32x16 G;
    if constexpr (!EXACT) {
      G = score_tile<D, NP>([&](int p, int s) { return row_op(dr + p * PS + 16 * s); },
                            [&](int p, int s) { return vop[p][s]; },
                            [](bf16x8 x, bf16x8 y, f32x16 c) { return mfma16(y, x, c); });
    } else {
#pragma unroll
      for (int e = 0; e < 16; ++e) G[e] = 0.f;
      const RowRead<D> rv(a.v + slice, jw, T, l32, half * (D / 2));
      const RowRead<D> rd(dos, i0, T, l32, half * (D / 2));
#pragma unroll 4
      for (int s = 0; s < D / 2; ++s) G = mfma32(rv.at(0, s), rd.at(0, s), G);
    }
    // some pair of the tile is not valid: key j is valid for this lane's
    // query i iff j <= jlim
    const bool edge = (a.causal & (jw + 31 > i0)) | (i0 + 32 > T) | (jw + 32 > T);
    const int i = i0 + l32;
    const int jlim = i < T ? (a.causal ? i : T - 1) : -1;
    float P[16], dS[16];
    if constexpr (EXPW) {
      // u holds the forward's fp32 exponential e (bf16-rounded for
      // BF16-exp); dz = gamma e (softmax; FP8-exp: the fp32
      // exponential's derivative through an identity rounding), BF16-exp
      // the backward of its casts, bf16(bf16(gamma) w)
      if (edge) {
#pragma unroll
        for (int r = 0; r < 16; ++r) u[r] = jw + krel(r, half) <= jlim ? u[r] : 0.f;
      }
      const float invWf = r1[3], invWX = r2[0], negDXW = r2[1];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float e = u[r];
        const float wf = RECON == REC_FP8EXP ? exp_weight_of<RECON>(e) : e;
        const float gamma = fmaf(G[r], invWX, negDXW);
        dS[r] = RECON == REC_BF16EXP ? bf16_rne(mul_or_0(bf16_rne(gamma), e))
                                          : mul_or_0(gamma, e);
        P[r] = wf * invWf;
        ps += dS[r];
      }
    } else {
      // a position whose weight is 0 (the FWM tail; below the argmin; minus
      // infinity) where the key is not valid
      constexpr float none = CALIB == CAL_FWM ? -1.f : CALIB == CAL_MINMAX ? -2.f : -INFINITY;
      if constexpr (COMPACT) {
        const uint32_t word[4] = {cw.x, cw.y, cw.z, cw.w};
#pragma unroll
        for (int r = 0; r < 16; ++r)  // r + up / 2, the tail -1/2
          u[r] = fmaf((float)((word[r >> 2] >> (8 * (r & 3))) & 0xFFu), 0.5f, -0.5f);
      }
      if (edge) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const bool valid = jw + krel(r, half) <= jlim;
          u[r] = valid ? u[r] : none;
          if constexpr (minmax) G[r] = valid ? G[r] : 0.f;  // (for pm)
        }
      }
      // e' = e^{b_{r+1}} / W from one exponential (RR_B1LW): P is e' or
      // e' e^{-h} (LERP: the chord between them), dS = (g c1 + c0) e'
      const float b1lw = r3[1], c1 = r3[2], c0 = r3[3];
      const float hl = minmax ? r0[3] : a.ghl, emh = minmax ? r1[1] : a.gemh;
      const float invWf = r1[3], invWX = r2[0], negDXW = r2[1], dcoef = r1[2];
      const float Wf = minmax ? 1.f / invWf : 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float rf = floorf(u[r]);
        if constexpr (!COMPACT) rf = fminf(minmax ? fmaxf(rf, 0.f) : rf, Kf - 1.f);
        float arg = fmaf(rf, hl, b1lw);
        if constexpr (CALIB == CAL_FWM) arg = u[r] < 0.f ? -INFINITY : arg;
        if constexpr (minmax) arg = u[r] < -1.f ? -INFINITY : arg;
        const float Ep = __builtin_amdgcn_exp2f(arg);
        const float Elp = Ep * emh;
        float t01 = u[r] - rf;
        if constexpr (CALIB == CAL_RESOLVED) t01 = __builtin_amdgcn_fmed3f(t01, 0.f, 1.f);
        float wLp = 0.f;
        if constexpr (!nearest || minmax) wLp = fmaf(t01, Ep - Elp, Elp);
        P[r] = nearest ? (t01 >= 0.5f ? Ep : Elp) : wLp;
        dS[r] = mul_or_0(fmaf(G[r], c1, c0), Ep);
        ps += dS[r];
        if (want_cm) {
          // dw^L/dM = X - w^L - Delta u / K, X = (r w^L + t e^{b_{r+1}}) / K,
          // on the unscaled weights
          const float Eu = Ep * Wf, wL = wLp * Wf;
          const float gamma = fmaf(G[r], invWX, negDXW);
          const float Delta = Eu * dcoef;
          const float uc = rf + t01;
          const float X = fmaf(rf, wL, t01 * Eu) * invK;
          pm += gamma * (X - wL - Delta * uc * invK);
        }
      }
    }
    // dS to its scratch tile, in the dQ product's operand type
    if constexpr (NP == 3) {
      tile_store(a.st.dS + tile, lane, dS);
    } else {
      // 2 KiB: element (lane l, register r) at (r/8)*512 + 8l + r%8
      uint16_t *dst = reinterpret_cast<uint16_t *>(a.st.dS) + tile + 8 * lane;
#pragma unroll
      for (int t2 = 0; t2 < 2; ++t2) {
        bf16x8 w[1];
        to_pieces<1>(reinterpret_cast<const float(&)[8]>(dS[8 * t2]), w);
        *reinterpret_cast<u32x4 *>(dst + 512 * t2) = __builtin_bit_cast(u32x4, w[0]);
      }
    }
    const int tb2 = tr_base<D>(lane);
    // (one piece: dS takes P's place in LDS before the first product, whose MFMAs
    // its reads then run under; B4 H16 T2048 d128 backward, this order / the other:
    // FWM Nearest 395 / 396 us, MinMax LERP 529 / 519, MinMax Nearest 682 / 690.
    // With three pieces the 24 more registers cost more than that)
    bf16x8 x[2][NP], xd[2][NP];
    if constexpr (EXACT) {
      product32(P, dos, i0, dva);
      product32(dS, qs, i0, dka);
    } else if constexpr (NP == 1) {
      put_tile(P);
      get_op(0, x[0]);
      get_op(1, x[1]);
      put_tile(dS);
      get_op(0, xd[0]);
      get_op(1, xd[1]);
      product(x, dOb + tb2, dva);
      product(xd, Qb + tb2, dka);
    } else {
      put_tile(P);
      get_op(0, x[0]);
      get_op(1, x[1]);
      product(x, dOb + tb2, dva);
      put_tile(dS);
      get_op(0, x[0]);
      get_op(1, x[1]);
      product(x, Qb + tb2, dka);
      dsr.add(dS);
    }
  };

  if (nt > 0) {
    fq.fetch(qs, qstart, T, tid);
    fd.fetch(dos, qstart, T, tid);
    fetch_rec(qstart);
  }
  for (int t = 0; t < nt; ++t) {
    const int i0 = qstart + t * BQ;
    uint16_t *Qb = Tl[t & 1], *dOb = Qb + St::SIZE;
    fq.stash(Qb, tid);
    fd.stash(dOb, tid);
    lds_barrier();
    if (t > 0) flush(t - 1);
    fq.fetch(qs, i0 + BQ, T, tid);
    fd.fetch(dos, i0 + BQ, T, tid);

    float ps = 0.f, pm = 0.f;
    if ((jw < T) & !(a.causal & (jw > i0 + 31))) {
      // (padding lanes of the last tile hold row T - 1's record)
      bool exact = false;
      if constexpr (NP == 3) exact = vout || __any(signbit(r3[0]));
      if constexpr (NP == 3)
        if (exact) tile_as(i0, Qb, dOb, ps, pm, std::true_type{});
      if (!exact) tile_as(i0, Qb, dOb, ps, pm, std::false_type{});
    }
    fetch_rec(i0 + BQ);  // the next tile's (past the last row: clamped)
    ps += __shfl_xor(ps, 32);
    pm += __shfl_xor(pm, 32);
    if (half == 0) {
      float *pp = Part[t & 1];
      pp[(wave * 32 + l32) * 2] = ps;
      pp[(wave * 32 + l32) * 2 + 1] = pm;
    }
  }
  if (nt == 0) return;  // a part without a tile has nothing to add
  lds_barrier();
  flush(nt - 1);
  if constexpr (NP == 3) {
    // dS out of range of the pieces: the wave's dK again on the fp32 MFMA, from the
    // dS tiles it stored
    if (dsr.out()) {
      __threadfence();
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int e = 0; e < 16; ++e) dka[c][e] = 0.f;
      const int key = 256 * (l32 >> 3) + 128 * ((l32 >> 2) & 1) + (l32 & 3);
#pragma unroll 1
      for (int i0 = qstart; i0 < qstart + nt * BQ; i0 += BQ) {
        if (a.causal & (jw > i0 + 31)) continue;
        const float *x = a.st.dS + ds_tile(bh, i0 / 32, jw / 32, nq, a.causal) * 1024 + key;
        const RowRead<D> rq(qs, i0, T, half, l32);
#pragma unroll 1
        for (int e = 0; e < 16; ++e) {
          const float xv = x[4 * (2 * e + half)];
#pragma unroll
          for (int c = 0; c < NC; ++c) dka[c] = mfma32(xv, rq.at(2 * e, 32 * c), dka[c]);
        }
      }
    }
  }
  // write dV, dK (lane -> column, register -> key)
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int j = jw + krel(r, half);
      if (j < T && 32 * c + l32 < D) {
        const size_t e = slice + (size_t)j * D + 32 * c + l32;
        if (a.qsplit > 1) {  // parts of the query range add up (zeroed by bwd_pre)
          atomicAdd((a.fold && qpart > 1 ? a.dq : a.dv) + e, dva[c][r]);
          atomicAdd(a.dk + e, a.scale * dka[c][r]);
        } else {
          if (NP == 1 && a.dv16) a.dv16[e] = (uint16_t)(__float_as_uint(bf16_rne(dva[c][r])) >> 16);
          else a.dv[e] = dva[c][r];
          a.dk[e] = a.scale * dka[c][r];
        }
      }
    }
}

// ---------------------------------------------------------------------------
// dQ = scale * (dS K + calibration terms). One workgroup = 2 QG waves = QG
// consecutive 32-query tiles of one (b,h) times two key halves (QG = 2 for
// d <= 64, 4 for d = 128): keys stream in chunks of 64 (one 32-key tile per
// half), staged row-major in bf16 pieces and read through transposing reads;
// a lane's own dS values are the A operand (split into pieces, or the bf16
// tile as it is). The kernel is bound by the latency and bandwidth of the dS
// tiles: each wave fetches its own two steps ahead, in two fixed register sets
// (loop unrolled by two), and one staging buffer leaves room for four
// workgroups per CU. The key halves' partial sums are added through LDS before
// the calibration epilogue.
template <typename TI, int D, int QG>
__global__ __launch_bounds__(128 * QG, (DqShape<TI, D>::OCC)) void bwd_dq_kernel(BwdArgsT<TI> a) {
  constexpr int NP = Pieces<TI>::N, NC = D >= 32 ? D / 32 : 1;
  constexpr int NT = 128 * QG;  // threads: QG query tiles x 2 key halves
  using St = Stage<D, 64, NT, TI>;
  constexpr int RS = St::RS, PS = St::PS, RED = QG * NC * 16 * 64 * 2;
  __shared__ __attribute__((aligned(16))) uint16_t Ks[St::SIZE > RED ? St::SIZE : RED];
  __shared__ int Bad[2 * QG];

  const int tid = threadIdx.x;
  const int lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // query tile pq of the QG and key half kh; key half 1 takes the query
  // tiles in reverse order, so that (QG = 4) the two waves of a SIMD (w and
  // w + 4) own query tiles pq and 3 - pq and their causal key ranges add up
  // alike
  const int kh = wave / QG, pq = kh ? QG - 1 - (wave % QG) : (wave % QG);
  const int T = a.T;
  const int nq = (T + 31) / 32;
  const int npq = (nq + QG - 1) / QG;
  const int bh = blockIdx.x % a.BH;
  // work item -> query group g (heaviest first) and its key piece sp
  int item = (int)(blockIdx.x / a.BH), g = npq - 1;
  while (item >= dq_pieces(g, T, a.causal, a.dq_piece, QG))
    item -= dq_pieces(g--, T, a.causal, a.dq_piece, QG);
  const int sp = item;
  const int nch = dq_chunks(g, T, a.causal, QG);
  const int c0 = a.dq_piece > 0 ? sp * a.dq_piece : 0;
  const int c1 = a.dq_piece > 0 ? min(nch, c0 + a.dq_piece) : nch;
  const int qt = QG * g + pq;
  const bool live = qt < nq;
  const int qtc = live ? qt : nq - 1;
  const size_t slice = (size_t)bh * T * D;
  const TI *ks = a.k + slice;
  const int nstep = c1 - c0;  // chunks of the piece
  const int ktmine = a.causal ? qtc : nq - 1;  // this wave's last key tile
  // this wave's tile of the piece's chunk p is kt = 2 (c0 + p) + kh; it is
  // used iff p < npw
  const int npw = !live || ktmine < kh ? 0 : max(0, min(c1, (ktmine - kh) / 2 + 1) - c0);
  const bool minmax = a.calib == CAL_MINMAX;

  f32x16 acc[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[c][e] = 0.f;

  St fk;
  auto fetch_k = [&](int p) { fk.fetch(ks, (c0 + min(p, nstep - 1)) * 64, T, tid); };
  // a dS tile: 16 fp32 per lane, or 16 bf16
  constexpr int ND = NP == 3 ? 4 : 2;
  u32x4 dA[ND], dB[ND];
  auto fetch_d = [&](int p, u32x4 (&dx)[ND]) {
    const int kt = min(2 * (c0 + min(p, nstep - 1)) + kh, ktmine);  // past this wave's row: unused
    const float *tile = a.st.dS + ds_tile(bh, qtc, kt, nq, a.causal) * 1024;
#pragma unroll
    for (int e = 0; e < ND; ++e)
      dx[e] = NP == 3 ? *reinterpret_cast<const u32x4 *>(tile + 256 * e + 4 * lane)
                      : *reinterpret_cast<const u32x4 *>(
                            reinterpret_cast<const uint16_t *>(a.st.dS) + (tile - a.st.dS) +
                            512 * e + 8 * lane);
  };
  const uint16_t *kb = Ks + kh * 32 * RS + tr_base<D>(lane);
  PieceCheck check;  // of the K values that this thread staged
  GradRange dsr;  // of this wave's dS
  auto mma_step = [&](const u32x4 (&dx)[ND]) {
    if constexpr (NP == 3) {
      float x[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) x[r] = __uint_as_float(dx[r / 4][r % 4]);
      dsr.add(x);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      bf16x8 av[NP];
      if constexpr (NP == 3) {
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = __uint_as_float(dx[2 * t + e / 4][e % 4]);
        to_pieces<3>(x, av);
      } else {
        av[0] = as_op(dx[t]);
      }
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        bf16x8 bv[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) bv[p] = tr_op<RS>(kb + p * PS + 16 * t * RS + 32 * c);
        acc[c] = mma<NP>(av, bv, acc[c]);
      }
    }
  };
  if (a.fold) {
    // the parts of dV that bwd_main left in this workgroup's rows of dq
    constexpr int PER = 32 * QG * D / 4 / NT;
    f32x4 x[PER], y[PER];
    const size_t e0 = (size_t)g * 32 * QG * D;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const size_t e = min(e0 + 4 * (tid + u * NT), (size_t)T * D - 4);
      x[u] = load4(a.dq + slice + e);
      y[u] = load4(a.dv + slice + e);
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const size_t e = e0 + 4 * (tid + u * NT);
      if (e < (size_t)T * D) *reinterpret_cast<f32x4 *>(a.dv + slice + e) = y[u] + x[u];
    }
  }
  fetch_k(0);
  fetch_d(0, dA);
  fetch_d(1, dB);
  // the calibration epilogue's row statistics (lanes 0..31: one row each)
  // and the q rows of its dK scatter, loaded behind the first two chunks'
  // fetches (so the first stash does not wait for them) and landing during
  // the key loop (every stats field exists for every calibration)
  constexpr int NE = (D + 63) / 64;
  const int row = qt * 32 + l32;
  const size_t ridx = (size_t)bh * T + (row < T ? row : T - 1);
  const float rflag = a.st.rowrec[ridx * RR_COUNT + RR_FLAGS];
  const int rnmax = a.st.nmax[ridx], rnmin = a.st.nmin[ridx];
  const float rss = a.st.sself[ridx], rcM = a.st.cM[ridx];
  const int ramax = a.st.amax[ridx], ramin = a.st.amin[ridx];
  float qv[16][NE];  // rows qt*32 + 16 kh + u of q, column lane + 64 x
  auto load_qv = [&]() {
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int qrow = qt * 32 + 16 * kh + u;
      const int qr = qrow < T ? qrow : T - 1;
#pragma unroll
      for (int x = 0; x < NE; ++x) {
        const int n = lane + 64 * x;
        qv[u][x] = load1(a.q + slice + (size_t)qr * D + (n < D ? n : 0));
      }
    }
  };
  // (d = 128: the 32 more registers would cost the key loop; loaded at the end)
  if constexpr (NE == 1) load_qv();
  auto step = [&](int p, u32x4 (&dx)[ND]) {
    if (p > 0) lds_barrier();
    fk.stash(Ks, tid, &check);
    fetch_k(p + 1);
    lds_barrier();
    if (p < npw) mma_step(dx);
    fetch_d(p + 2, dx);
  };
  for (int p = 0; p < nstep; p += 2) {
    step(p, dA);
    if (p + 1 >= nstep) break;
    step(p + 1, dB);
  }
  if constexpr (NP == 3) {
    const bool out = __any(check.bad());
    if (lane == 0) Bad[wave] = out;
  }
  // key half 1 hands its partial sums to key half 0
  __syncthreads();
  if constexpr (NP == 3) {
    // values out of range of the pieces in the K chunks or in this wave's dS, or a
    // row of dO or q that is marked (its own dS may be): the wave's product again
    // on the fp32 MFMA, its operands from memory
    if (any_flag<2 * QG>(Bad) || dsr.out() || __any(signbit(rflag))) {
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[c][e] = 0.f;
#pragma unroll 1
      for (int p = 0; p < npw; ++p) {
        const int kt = 2 * (c0 + p) + kh;
        const RowRead<D> rk(ks, kt * 32, T, 4 * half, l32);
        const float *x = a.st.dS + ds_tile(bh, qtc, kt, nq, a.causal) * 1024 + 4 * lane;
#pragma unroll 1
        for (int r = 0; r < 16; ++r) {
          const float xv = x[256 * (r >> 2) + (r & 3)];
#pragma unroll
          for (int c = 0; c < NC; ++c) acc[c] = mfma32(xv, rk.at(krel0(r), 32 * c), acc[c]);
        }
      }
    }
  }
  {
    float *red = reinterpret_cast<float *>(Ks) + pq * (NC * 16 * 64) + lane;
    if (kh == 1) {
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int e = 0; e < 16; ++e) red[(c * 16 + e) * 64] = acc[c][e];
    }
    __syncthreads();
    if (kh == 0) {
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[c][e] += red[(c * 16 + e) * 64];
    }
  }
  if (!live) return;  // no barrier below

  // calibration terms of rows with unique extrema (lanes 0..31: one row each)
  bool ok = false;
  float cMt = 0.f, cm = 0.f;
  int am = 0, an = 0;
  const bool cal = sp == 0 && grad_channels(a.grad);  // piece 0 adds them
  if (cal && row < T && rflag == 0.f) {
    const int nmin = minmax ? rnmin : 1;
    ok = (rnmax == 1) & (nmin == 1);
    cMt = minmax ? rcM : -rss;
    cm = minmax ? -(rss + cMt) : 0.f;
    if (!grad_keep_max(a.grad)) cMt = 0.f;
    if (!grad_keep_min(a.grad)) cm = 0.f;
    am = ramax;
    an = minmax ? ramin : am;
  }
  if (!ok) { cMt = 0.f; cm = 0.f; am = 0; an = 0; }
  // dQ rows (key half 0): register e holds query krel(e, half), lane column
  // 32c + l32. The k rows of the calibration terms are gathered for EB rows
  // at a time before their dQ stores (stores to dq could alias k, so a load
  // after a store waits for it: one memory round trip per batch, not per
  // row); the argmin term exists for MinMax only (cm = 0 otherwise)
  constexpr int EB = D <= 32 ? 16 : (D == 64 ? 8 : 4);
  if (kh == 0) {
#pragma unroll
  for (int e0 = 0; e0 < 16; e0 += EB) {
    float kM[EB][NC] = {}, km[EB][NC] = {};
    if (cal) {
#pragma unroll
      for (int b = 0; b < EB; ++b) {
        const int src = krel(e0 + b, half);
        const int iam = __shfl(am, src);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const int n = 32 * c + l32;
          kM[b][c] = load1(ks + (size_t)iam * D + (n < D ? n : 0));
        }
      }
      if (minmax) {
#pragma unroll
        for (int b = 0; b < EB; ++b) {
          const int ian = __shfl(an, krel(e0 + b, half));
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            const int n = 32 * c + l32;
            km[b][c] = load1(ks + (size_t)ian * D + (n < D ? n : 0));
          }
        }
      }
    }
#pragma unroll
    for (int b = 0; b < EB; ++b) {
      const int e = e0 + b;
      const int src = krel(e, half);
      const float fM = __shfl(cMt, src), fm = __shfl(cm, src);
      const int qrow = qt * 32 + src;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int n = 32 * c + l32;
        float v = acc[c][e];
        v = fmaf(fM, kM[b][c], v);
        v = fmaf(fm, km[b][c], v);
        if (qrow < T && n < D) {
          if (a.dq_piece > 0) atomicAdd(a.dq + slice + (size_t)qrow * D + n, a.scale * v);
          else a.dq[slice + (size_t)qrow * D + n] = a.scale * v;
        }
      }
    }
  }
  }
  // scatter of the calibration terms onto the argmax/argmin keys of dK
  // (each key half takes 16 rows, their q preloaded; piece 0 only)
  // the deterministic backward gathers these per key instead: one record
  // per row for it
  if (a.det && grad_channels(a.grad) && kh == 0 && half == 0 && row < T)
    put_calib_record(a.st.part, ridx, ok, minmax, am, an, cMt * a.scale, cm * a.scale);
  if (cal && !a.det) {
    if constexpr (NE > 1) load_qv();
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int rr = 16 * kh + u;
      if (!__shfl(ok ? 1 : 0, rr)) continue;  // wave-uniform
      const float fM = __shfl(cMt, rr) * a.scale, fm = __shfl(cm, rr) * a.scale;
      const int iam = __shfl(am, rr), ian = __shfl(an, rr);
#pragma unroll
      for (int x = 0; x < NE; ++x) {
        const int n = lane + 64 * x;
        if (n < D) {
          atomicAdd(a.dk + slice + (size_t)iam * D + n, fM * qv[u][x]);
          if (minmax) atomicAdd(a.dk + slice + (size_t)ian * D + n, fm * qv[u][x]);
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Rows with tied extrema of one 32-row block rb of slice bh, by one wave.
template <int D, typename TI>
__device__ __forceinline__ void tie_rows(const BwdArgsT<TI> &a, int bh, int rb, int lane) {
  const int half = lane >> 5, l32 = lane & 31;
  const int T = a.T;
  const int i = rb * 32 + l32;
  const bool minmax = a.calib == CAL_MINMAX;
  const size_t slice = (size_t)bh * T * D;
  const size_t ridx = (size_t)bh * T + (i < T ? i : T - 1);
  bool tierow = false;
  float M = 0.f, m = 0.f, coefM = 0.f, coefm = 0.f;
  if (i < T && a.st.rowrec[ridx * RR_COUNT + RR_FLAGS] == 0.f) {
    const int nmax = a.st.nmax[ridx];
    const int nmin = minmax ? a.st.nmin[ridx] : 1;
    tierow = (nmax > 1) | (nmin > 1);
    const float ss = a.st.sself[ridx];
    const float cMt = minmax ? a.st.cM[ridx] : -ss;
    const float cm = minmax ? -(ss + cMt) : 0.f;
    M = a.st.M[ridx];
    m = minmax ? a.st.m[ridx] : M;
    coefM = grad_keep_max(a.grad) ? cMt / (float)nmax : 0.f;
    coefm = grad_keep_min(a.grad) ? cm / (float)nmin : 0.f;
  }
  if (!__any(tierow)) return;
  // the row's scores with the canonical sub-tile of the input type
  ScoreOp<TI, D> qop;
  qop.load(a.q + slice, i < T ? i : T - 1, T, half);
  auto tile_scores = [&](int js) -> f32x16 {
    ScoreOp<TI, D> kop;
    kop.load(a.k + slice, js + l32, T, half);
    return ScoreOp<TI, D>::tile(kop, qop);
  };
  const int kend = a.causal ? min(T, rb * 32 + 32) : T;
  for (int js = 0; js < kend; js += 32) {
    const f32x16 acc = tile_scores(js);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int j = js + krel(r, half);
      const bool valid = tierow & (j < T) & (!a.causal | (j <= i));
      const float s = acc[r] * a.scale;
      const bool hitM = valid & (s == M);
      const bool hitm = valid & minmax & (s == m);
      const float coef = hitM ? coefM : (hitm ? coefm : 0.f);
      uint64_t mask = __ballot(hitM | hitm);
      while (mask) {
        const int src = __ffsll((unsigned long long)mask) - 1;
        mask &= mask - 1;
        const float cf = __shfl(coef, src) * a.scale;
        const int isrc = rb * 32 + (src & 31);
        const int jsrc = js + krel(r, src >> 5);
        for (int e = lane; e < D; e += 64) {
          const float dqv = cf * load1(a.k + slice + (size_t)jsrc * D + e);
          const float dkv = cf * load1(a.q + slice + (size_t)isrc * D + e);
          if (a.det) {
            // one wave per slice: element e is always this lane's, in order
            a.dq[slice + (size_t)isrc * D + e] += dqv;
            a.dk[slice + (size_t)jsrc * D + e] += dkv;
          } else {
            atomicAdd(a.dq + slice + (size_t)isrc * D + e, dqv);
            atomicAdd(a.dk + slice + (size_t)jsrc * D + e, dkv);
          }
        }
      }
    }
  }
}

// Ties: one wave per 32-row block, or in the deterministic backward one wave
// per (b, h) slice taking its row blocks in order (so that each dK row of the
// slice receives its tie terms from one wave, in a fixed order).
template <int D, typename TI>
__global__ __launch_bounds__(256) void bwd_ties_kernel(BwdArgsT<TI> a) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nrb = (a.T + 31) / 32;
  const size_t gw = (size_t)blockIdx.x * 4 + wave;
  if (a.det) {
    if (gw >= (size_t)a.BH) return;
    // which row blocks hold a tied row: 256 rows per round of loads
    const int T = a.T, bh = (int)gw;
    const bool minmax = a.calib == CAL_MINMAX;
    for (int r0 = 0; r0 < T; r0 += 256) {
      bool tie[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int i = r0 + 64 * c + lane;
        const size_t ridx = (size_t)bh * T + (i < T ? i : T - 1);
        const int nmin = minmax ? a.st.nmin[ridx] : 1;
        tie[c] = (i < T) & ((a.st.nmax[ridx] > 1) | (nmin > 1)) &
                 (a.st.rowrec[ridx * RR_COUNT + RR_FLAGS] == 0.f);
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const uint64_t m = __ballot(tie[c]);
        const int rb = (r0 + 64 * c) / 32;
        if (m & 0xffffffffull) tie_rows<D, TI>(a, bh, rb, lane);
        if (m >> 32) tie_rows<D, TI>(a, bh, rb + 1, lane);
      }
    }
  } else {
    if (gw >= (size_t)a.BH * nrb) return;
    tie_rows<D, TI>(a, (int)(gw / nrb), (int)(gw % nrb), lane);
  }
}

// Deterministic backward: S_self (and cM under MinMax) of every row as the
// sum of its key blocks' partials, in key-block order (causal: the blocks
// at or below the row's own).
template <typename TI>
__global__ __launch_bounds__(256) void row_sums_kernel(BwdArgsT<TI> a) {
  const size_t R = (size_t)a.BH * a.T;
  const size_t ridx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (ridx >= R) return;
  const int i = (int)(ridx % (size_t)a.T);
  const int nkb = (a.T + 127) / 128;
  const int kend = a.causal ? i / 128 + 1 : nkb;
  const bool minmax = a.calib == CAL_MINMAX;
  float s = 0.f, mm = 0.f;
  for (int kb = 0; kb < kend; ++kb) {
    s += a.st.part[(size_t)kb * R + ridx];
    if (minmax) mm += a.st.part[(size_t)(nkb + kb) * R + ridx];
  }
  a.st.sself[ridx] = s;
  if (minmax) a.st.cM[ridx] = mm;
}

// Deterministic backward: the calibration terms of the rows with unique
// extrema (the ones bwd_dq scatters otherwise), gathered onto dK. bwd_dq
// leaves one record per row in st.part (put_calib_record); one wave per 32
// keys of a slice scans the records in row order (causal: from its first
// key on), collects scale cM_i q_i on key amax_i and scale cm_i q_i on key
// amin_i in LDS, then adds each key's sum to its dK row.
template <int D, typename TI, int NW>
__global__ __launch_bounds__(64 * NW) void calib_gather_kernel(BwdArgsT<TI> a) {
  constexpr int NE = (D + 63) / 64;
  constexpr int GB = 16;  // hit rows whose q rows are loaded together
  // NW waves: wave w takes the 256-row rounds w, w + NW, ... and the keys
  // 32 w / NW onwards of the final sum
  __shared__ float acc[NW][32 * D];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int T = a.T, nkt = (T + 31) / 32;
  const int bh = blockIdx.x / nkt, j0 = (blockIdx.x % nkt) * 32;
  const size_t slice = (size_t)bh * T * D;
  const f32x4 *rec = reinterpret_cast<const f32x4 *>(a.st.part) + (size_t)bh * T;
  float *accw = acc[w];
  for (int e = lane; e < 32 * D; e += 64) accw[e] = 0.f;
  __syncthreads();
  const int ibeg = a.causal ? j0 : 0;
  for (int r0 = ibeg + 256 * w; r0 < T; r0 += 256 * NW) {
    // the records of 256 rows in one round of loads
    f32x4 rc[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int i = r0 + 64 * c + lane;
      rc[c] = rec[i < T ? i : T - 1];
      if (i >= T) rc[c] = f32x4{-1.f, 0.f, -1.f, 0.f};
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int kMl = (int)rc[c][0] - j0, kml = (int)rc[c][2] - j0;
      const bool hM = rc[c][0] >= 0.f && kMl >= 0 && kMl < 32;
      const bool hm = rc[c][2] >= 0.f && kml >= 0 && kml < 32;
      uint64_t mask = __ballot(hM | hm);
      const int i0 = r0 + 64 * c;
      // the hit rows in order, GB at a time: their q rows are loaded
      // together, then added one after the other
      while (mask) {
        int src[GB];
#pragma unroll
        for (int b = 0; b < GB; ++b) {
          src[b] = mask ? __ffsll((unsigned long long)mask) - 1 : -1;
          mask &= mask ? mask - 1 : 0;
        }
        // (unconditional loads from clamped addresses, so that they are all
        // in flight together; unused slots are zeroed after)
        float qv[GB][NE];
#pragma unroll
        for (int b = 0; b < GB; ++b) {
          const TI *qr = a.q + slice + (size_t)(i0 + (src[b] >= 0 ? src[b] : 0)) * D;
#pragma unroll
          for (int x = 0; x < NE; ++x) {
            const int n = lane + 64 * x;
            const float t = load1(qr + (n < D ? n : 0));
            qv[b][x] = (src[b] >= 0 && n < D) ? t : 0.f;
          }
        }
        // per channel, the batch's consecutive hits on one key are summed in
        // registers (in row order) and that run added to the key's LDS row
        // once: keys that hold the argmax of many rows do not serialize on
        // one LDS address
#pragma unroll
        for (int ch = 0; ch < 2; ++ch) {
          const int kl = ch == 0 ? (hM ? kMl : -1) : (hm ? kml : -1);
          const float fl = rc[c][ch == 0 ? 1 : 3];
          int cur = -1;
          float run[NE];
#pragma unroll
          for (int x = 0; x < NE; ++x) run[x] = 0.f;
#pragma unroll
          for (int b = 0; b < GB; ++b) {
            if (src[b] < 0) break;  // wave-uniform
            const int key = __shfl(kl, src[b]);
            if (key < 0) continue;
            const float f = __shfl(fl, src[b]);
            if (key != cur) {
              if (cur >= 0) {
#pragma unroll
                for (int x = 0; x < NE; ++x)
                  if (lane + 64 * x < D) accw[cur * D + lane + 64 * x] += run[x];
              }
              cur = key;
#pragma unroll
              for (int x = 0; x < NE; ++x) run[x] = 0.f;
            }
#pragma unroll
            for (int x = 0; x < NE; ++x) run[x] = fmaf(f, qv[b][x], run[x]);
          }
          if (cur >= 0) {
#pragma unroll
            for (int x = 0; x < NE; ++x)
              if (lane + 64 * x < D) accw[cur * D + lane + 64 * x] += run[x];
          }
        }
      }
    }
  }
  __syncthreads();
  // the waves' sums in wave order onto the dK rows; wave w takes KPW keys
  // (their rows loaded together, then stored)
  constexpr int KPW = 32 / NW;
  float dk[KPW][NE];
#pragma unroll
  for (int t = 0; t < KPW; ++t)
#pragma unroll
    for (int x = 0; x < NE; ++x) {
      const int n = lane + 64 * x;
      const int j = j0 + KPW * w + t < T ? j0 + KPW * w + t : T - 1;
      dk[t][x] = a.dk[slice + (size_t)j * D + (n < D ? n : 0)];
    }
#pragma unroll
  for (int t = 0; t < KPW; ++t)
#pragma unroll
    for (int x = 0; x < NE; ++x) {
      const int n = lane + 64 * x, jj = KPW * w + t;
      if ((j0 + jj < T) & (n < D)) {
        float sum = acc[0][jj * D + n];
#pragma unroll
        for (int v = 1; v < NW; ++v) sum += acc[v][jj * D + n];
        a.dk[slice + (size_t)(j0 + jj) * D + n] = dk[t][x] + sum;
      }
    }
}

// ---------------------------------------------------------------------------
// P1 (App. B, Detach): each detached row of dS minus its mean over the row's
// n_i valid keys, applied to dQ and dK as rank-1 corrections,
//   dQ_i -= scale * mean_i * sum_{j valid for i} k_j
//   dK_j -= scale * sum_{i: j valid for i} mean_i q_i,   mean_i = S_self_i / n_i
// (dV has no calibration term). One workgroup per (b,h) and 64 columns:
// four row segments scan in parallel and are combined through LDS.
template <int D, typename TI>
__global__ __launch_bounds__(256) void bwd_p1_kernel(BwdArgsT<TI> a) {
  constexpr int NCB = (D + 63) / 64;
  __shared__ float part[2][4][64];
  const int tid = threadIdx.x, cl = tid & 63, seg = tid >> 6;
  const int bh = blockIdx.x / NCB, cb = blockIdx.x % NCB;
  const int col = cb * 64 + cl;
  const bool cok = col < D;
  const int T = a.T;
  const int L = (T + 3) / 4;
  const int r0 = min(T, seg * L), r1 = min(T, r0 + L);
  const size_t slice = (size_t)bh * T * D;
  const float *ss = a.st.sself + (size_t)bh * T;
  auto mean = [&](int i) { return ss[i] / (float)(a.causal ? i + 1 : T); };
  const int cc = cok ? col : 0;
  float ks = 0.f, qs = 0.f;
  for (int i = r0; i < r1; ++i) {
    ks += load1(a.k + slice + (size_t)i * D + cc);
    qs += mean(i) * load1(a.q + slice + (size_t)i * D + cc);
  }
  part[0][seg][cl] = ks;
  part[1][seg][cl] = qs;
  __syncthreads();
  float kpre = 0.f, qsuf = 0.f, ktot = 0.f, qtot = 0.f;
#pragma unroll
  for (int s2 = 0; s2 < 4; ++s2) {
    const float kk = part[0][s2][cl], qq = part[1][s2][cl];
    ktot += kk;
    qtot += qq;
    if (s2 < seg) kpre += kk;
    if (s2 > seg) qsuf += qq;
  }
  if (!cok) return;
  for (int i = r0; i < r1; ++i) {
    kpre += load1(a.k + slice + (size_t)i * D + col);
    a.dq[slice + (size_t)i * D + col] -= a.scale * mean(i) * (a.causal ? kpre : ktot);
  }
  for (int j = r1 - 1; j >= r0; --j) {
    qsuf += mean(j) * load1(a.q + slice + (size_t)j * D + col);
    a.dk[slice + (size_t)j * D + col] -= a.scale * (a.causal ? qsuf : qtot);
  }
}

#if KIA_HEAD == 64  // no head dimension: once
// ---------------------------------------------------------------------------
// Score-gradient decomposition export: g_self dense from the dS scratch
// (fp32 tiles, or bf16 tiles of the bf16 variant) and the row sums of the
// two extremum channels. One wave per (b,h, 32-query tile).
__global__ __launch_bounds__(256) void score_grad_kernel(GradArgs a) {
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6, half = lane >> 5, l32 = lane & 31;
  const int T = a.T;
  const int nq = (T + 31) / 32;
  const size_t gw = (size_t)blockIdx.x * 4 + wave;
  if (gw >= (size_t)a.BH * nq) return;
  const int bh = (int)(gw / nq), qt = (int)(gw % nq);
  const int i = qt * 32 + l32;
  const bool minmax = a.calib == CAL_MINMAX;
  if (half == 0 && i < T) {
    const size_t ridx = (size_t)bh * T + i;
    const bool degen = a.st.rowrec[ridx * RR_COUNT + RR_FLAGS] != 0.f;
    const float s = a.st.sself[ridx];
    const float cMv = degen ? 0.f : (minmax ? a.st.cM[ridx] : -s);
    a.cM[ridx] = cMv;
    a.cm[ridx] = (degen || !minmax) ? 0.f : -(s + cMv);
  }
  for (int kt = 0; kt < nq; ++kt) {
    const bool stored = !a.causal || kt <= qt;
    float v[16];
    if (stored) {
      const size_t tile = ds_tile(bh, qt, kt, nq, a.causal) * 1024;
      if (a.bf16) {
        const uint16_t *src = reinterpret_cast<const uint16_t *>(a.st.dS) + tile + 8 * lane;
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = bf2f(src[512 * (r / 8) + r % 8]);
      } else {
        tile_load(a.st.dS + tile, lane, v);
      }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int j = kt * 32 + krel(r, half);
      if (i < T && j < T)
        a.g_self[((size_t)bh * T + i) * T + j] =
            (stored && (!a.causal || j <= i)) ? v[r] : 0.f;
    }
  }
}

#endif

// One head dimension per compilation (KIA_HEAD, set by the build).
#define KIA_MAIN_GRID(TI, D)                                                          \
  template __global__ void bwd_main_kernel<TI, D, CAL_MINMAX, REC_LERP>(BwdArgsT<TI>);    \
  template __global__ void bwd_main_kernel<TI, D, CAL_MINMAX, REC_NEAREST>(BwdArgsT<TI>); \
  template __global__ void bwd_main_kernel<TI, D, CAL_FWM, REC_LERP>(BwdArgsT<TI>);       \
  template __global__ void bwd_main_kernel<TI, D, CAL_FWM, REC_NEAREST>(BwdArgsT<TI>);    \
  template __global__ void bwd_main_kernel<TI, D, CAL_RESOLVED, REC_LERP>(BwdArgsT<TI>);  \
  template __global__ void bwd_main_kernel<TI, D, CAL_RESOLVED, REC_NEAREST>(BwdArgsT<TI>);
#define KIA_BWD_TI(TI, D)                                              \
  KIA_MAIN_GRID(TI, D)                                                 \
  template __global__ void bwd_pre_kernel<D, TI>(BwdArgsT<TI>);        \
  template __global__ void bwd_dq_kernel<TI, D, dq_tiles(D)>(BwdArgsT<TI>); \
  template __global__ void bwd_ties_kernel<D, TI>(BwdArgsT<TI>);       \
  template __global__ void bwd_p1_kernel<D, TI>(BwdArgsT<TI>);         \
  template __global__ void calib_gather_kernel<D, TI, 1>(BwdArgsT<TI>); \
  template __global__ void calib_gather_kernel<D, TI, 4>(BwdArgsT<TI>);
#define KIA_BWD(D)                                                                \
  KIA_BWD_TI(float, D)                                                            \
  KIA_BWD_TI(uint16_t, D)                                                         \
  template __global__ void bwd_main_kernel<float, D, CAL_FWM, REC_SOFTMAX>(BwdArgs); \
  template __global__ void bwd_main_kernel<float, D, CAL_FWM, REC_BF16EXP>(BwdArgs); \
  template __global__ void bwd_main_kernel<float, D, CAL_FWM, REC_FP8EXP>(BwdArgs);
KIA_BWD(KIA_HEAD)

#if KIA_HEAD == 64  // no head dimension: once
template __global__ void row_sums_kernel<float>(BwdArgs);
template __global__ void row_sums_kernel<uint16_t>(BwdArgs16);
#endif

}  // namespace kia
