// kia_device.hpp -- device building blocks shared by every K-interval
// attention kernel for gfx950 (CDNA4, wave64, bf16 MFMA 32x32x16 with fp32
// accumulation; fp32 scores on the fp32 MFMA 32x32x2).
//
// fp32 operands on the bf16 matrix unit. An fp32 value of 2^-100 to 2^126, or 0,
// is the exact sum of three bf16 pieces x = x0 + x1 + x2, each the nearest bf16
// of what is left (|x1| <= 2^-9 |x|, |x2| <= 2^-18 |x|; for other values see
// PieceCheck), and a product x y is taken as the six
// piece products down to 2^-18: x2 y0, x1 y1, x0 y2, x1 y0, x0 y1, x0 y0. The
// three that are left out are at most 2^-26 |x y| together, below the fp32
// rounding of one product. bf16 MFMA runs at 16 times the fp32 MFMA's rate, so
// six of them take 0.375 of its time, and unlike it they overlap with VALU
// work of the SIMD's other wave. Against 64 bits (N(0,1) operands, one 32x32
// tile, measured on the device): contraction length 64, 1.44e-7 (fp32 MFMA)
// and 4.6e-8 (the six products added smallest first); 128, 2.04e-7 and
// 6.2e-8; streamed over 512 with the six products of 16 terms at a time,
// 4.1e-7 and 3.4e-7. bf16 inputs are one piece and one product.
//
// Canonical score sub-tile. Every kernel that needs a score s_ij computes it
// with ScoreOp::tile(): a 32-key x 32-query block of S^T accumulated over d in
// one fixed order, by v_mfma_f32_32x32x2_f32 for fp32 inputs (d/2 steps of the
// terms s and d/2 + s, each a fused multiply-add) and v_mfma_f32_32x32x16_bf16
// for bf16 inputs, with the key block and the query block aligned to multiples
// of 32. The A operand is K (rows = keys), the B operand Q (columns = queries).
// Lane l (half h = l/32) feeds, at k-step s, K[key0 + l%32][h d/2 + s] and the
// same of Q (bf16: [16 s + 8 h + e], e = 0..7). Output register r of lane l holds
// S^T[key0 + krel(r, h)][query0 + l%32] with krel(r, h) = 8*(r/4) + 4*h + r%4.
// Same operands, same instruction sequence, same lane/register position: the fp32
// score of a pair is bit-identical wherever it is computed (both passes of the
// forward, the tie path and the debug exports), which the exact extremum ties and
// index decisions rely on.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace kia {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// CAL_RESOLVED: the tail-policy diagnostic (FWM's step tau/K and origin -tau,
// the grid continued below -tau with negative intervals, no zero tail)
enum { CAL_MINMAX = 0, CAL_FWM = 1, CAL_RESOLVED = 2 };
// K-interval reconstructions, then the exponential weight functions of the
// baselines: exact softmax (App. A) and the reduced-precision exponentials
// BF16-exp and FP8 (E4M3)-rounded exp (App. D). The latter three use only
// the row maximum (z = s - M) and no grid.
enum { REC_LERP = 0, REC_NEAREST = 1, REC_SOFTMAX = 2, REC_BF16EXP = 3, REC_FP8EXP = 4 };
__host__ __device__ constexpr bool is_exp_rec(int r) { return r >= REC_SOFTMAX; }
enum { STE_WEIGHT = 0, STE_PROB = 1 };

// Row record written by the backward's preprocessing (16 floats per row).
// RR_B1LW = b1l - log2 W: exp2(r hl + b1lw) = e^{b_{r+1}} / W, so the forward
// probability comes out of the exponential directly; RR_C1, RR_C0: gamma
// Delta = (g c1 + c0) e^{b_{r+1}} / W with c1 = dcoef W / W^X and
// c0 = -dcoef W D^X / W^X.
enum {
  RR_ALPHA = 0, RR_BETA, RR_MARGIN2, RR_HL, RR_B1L, RR_EMH, RR_DCOEF,
  RR_INVWF, RR_INVWX, RR_NEGDXW, RR_M, RR_m, RR_FLAGS, RR_B1LW, RR_C1, RR_C0,
  RR_COUNT = 16
};

// Device view of the caller's stats buffer (layout documented in kia.h).
struct Stats {
  float *M, *m, *W, *WL;
  int *amax, *amin, *nmax, *nmin;
  float *rowrec;  // [R][RR_COUNT]
  float *sself, *cM;
  float *OL;      // [R][d] or nullptr
  float *dS;      // backward scratch: dS in 32x32 tiles, 1024 floats each
  float *U;       // fp32 scores between the forward's passes, then its decisions, same tiles
  float *part;    // deterministic backward: row-sum partials [2][ceil(T/128)][R],
                  // then the calibration records [R][4] of the dK gather
};

// Deterministic backward: a row's calibration record for the dK gather, as
// the dQ kernel's epilogue decides it: {argmax key or -1, scale cM, argmin
// key or -1, scale cm} (-1: the row is not one with unique extrema, or the
// channel is not taken).
__device__ __forceinline__ void put_calib_record(float *part, size_t ridx, bool ok, bool minmax,
                                                 int am, int an, float fM, float fm) {
  reinterpret_cast<f32x4 *>(part)[ridx] =
      f32x4{ok ? (float)am : -1.f, fM, (ok && minmax) ? (float)an : -1.f, fm};
}

// The row sums of one 128-key block's score gradients (S_self, and cM under
// MinMax): added atomically, or, in the deterministic backward, stored as
// the block's partial for a sum in key-block order.
template <typename A>
__device__ __forceinline__ void put_row_sums(const A &a, int kb, size_t ridx, float s,
                                             float mm, bool minmax) {
  if (a.det) {
    const size_t R = (size_t)a.BH * a.T;
    const int nkb = (a.T + 127) / 128;
    a.st.part[(size_t)kb * R + ridx] = s;
    if (minmax) a.st.part[(size_t)(nkb + kb) * R + ridx] = mm;
  } else {
    atomicAdd(a.st.sself + ridx, s);
    if (minmax) atomicAdd(a.st.cM + ridx, mm);
  }
}

__device__ __forceinline__ f32x16 mfma32(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ int krel(int r, int half) {
  return 8 * (r >> 2) + 4 * half + (r & 3);
}

// Per-row constants of the fast index/weight evaluation.
//   u_fast = fma(acc, alpha, beta) approximates u (MinMax (K(s-m))/(M-m),
//   FWM K(s-M+tau)/tau) within margin2/2 (worst-case rounding bound x8);
//   E_{r+1} = exp2(r*hl + b1l) = e^{b_{r+1}}, E_r = E_{r+1} * emh (emh =
//   e^{-h}), Delta_r = E_{r+1} * dcoef (dcoef = (1 - e^{-h})/h).
// Degenerate MinMax rows (M - m <= 1e-12, App. A) map every key to u = K
// with all weights 1 and Delta = 0.
struct RowConst {
  float alpha, beta, margin2, hl, b1l, emh, dcoef;
  bool degen;
};

__device__ inline RowConst row_const(float M, float m, int K, int calib,
                                     float tau, float scale) {
  RowConst rc;
  const double Kd = (double)K;
  const double LOG2E = 1.4426950408889634074;
  double h, zlo;
  rc.degen = false;
  if (calib == CAL_MINMAX) {
    const double span = (double)M - (double)m;
    if (span <= 1e-12) {
      rc.degen = true;
      rc.alpha = 0.f; rc.beta = (float)K; rc.margin2 = 0.f;
      rc.hl = 0.f; rc.b1l = 0.f; rc.emh = 1.f; rc.dcoef = 0.f;
      return rc;
    }
    const double c = Kd / span;
    rc.alpha = (float)(c * (double)scale);
    rc.beta = (float)(-(double)m * c);
    const double A = fmax(fabs((double)M), fabs((double)m));
    rc.margin2 = (float)ldexp(3.0 * c * A + Kd, -20);
    h = span / Kd;
    zlo = (double)m - (double)M;
  } else {
    const double t = (double)tau;
    const double c = Kd / t;
    rc.alpha = (float)(c * (double)scale);
    rc.beta = (float)(Kd - (double)M * c);
    // FWM decides window keys only (|s| <= |M| + tau); the resolved grid
    // decides every key, down to m, where |u| reaches c (M - m) + K
    const double A = calib == CAL_RESOLVED
                         ? fmax(fabs((double)M), fabs((double)m)) + t + ((double)M - (double)m)
                         : fabs((double)M) + t;
    rc.margin2 = (float)ldexp(3.0 * c * A + 2.0 * Kd, -20);
    h = t / Kd;
    zlo = -t;
  }
  rc.hl = (float)(h * LOG2E);
  rc.b1l = (float)((zlo + h) * LOG2E);
  rc.emh = (float)exp(-h);
  rc.dcoef = (float)(-expm1(-h) / h);
  return rc;
}

// The grid constants the backward uses (hl, b1l, emh, dcoef of RowConst),
// in fp32 except the degenerate test, which must be the forward's
// (fp64 span <= 1e-12). A few ulp from row_const's fp64-derived values.
__device__ inline void grid_consts(float M, float m, int K, int calib, float tau,
                                   float &hl, float &b1l, float &emh, float &dcoef,
                                   bool &degen) {
  const float LOG2E = 1.44269504f;
  float h, zlo;
  degen = false;
  if (calib == CAL_MINMAX) {
    if ((double)M - (double)m <= 1e-12) {
      degen = true;
      hl = 0.f; b1l = 0.f; emh = 1.f; dcoef = 0.f;
      return;
    }
    zlo = m - M;
    h = -zlo / (float)K;
  } else {
    zlo = -tau;
    h = tau / (float)K;
  }
  hl = h * LOG2E;
  b1l = (zlo + h) * LOG2E;
  emh = expf(-h);
  dcoef = -expm1f(-h) / h;
}

// Exact index decision on the fp32 score s (fp64 expressions of kia.h).
__device__ __forceinline__ void exact_decision(float s, float M, float m, int K,
                                            int calib, float tau, float &rf,
                                            int &up, int &tail) {
#pragma clang fp contract(off)
  double u;
  tail = 0;
  if (calib == CAL_MINMAX) {
    u = ((double)K * ((double)s - (double)m)) / ((double)M - (double)m);
  } else if (calib == CAL_RESOLVED) {
    u = ((double)K * (((double)s - (double)M) + (double)tau)) / (double)tau;
  } else {
    const double a = ((double)s - (double)M) + (double)tau;
    if (a < 0.0) {
      tail = 1; rf = 0.f; up = 0;
      return;
    }
    u = ((double)K * a) / (double)tau;
  }
  double r = floor(u);
  if (r < 0.0 && calib != CAL_RESOLVED) r = 0.0;  // the resolved grid has no lower end
  if (r > (double)(K - 1)) r = (double)(K - 1);
  double t = u - r;
  if (t < 0.0) t = 0.0;
  if (t > 1.0) t = 1.0;
  rf = (float)r;
  up = t >= 0.5 ? 1 : 0;
}

// Index decisions of the 16 keys a lane holds in one score sub-tile, kept
// as one fp32 position u per key (r, t, l and the FWM tail are re-derived
// from u by key_of()). Fast path: u = fma(acc, alpha, beta). A key whose u
// lies within the rounding margin of an interior integer/half-integer
// (~1e-5 of keys) is decided by exact_decision() and its u is clamped into
// the interval of that decision (one key per lane per round), so that
// key_of() reproduces the exact decision and t stays within the margin.
template <int CALIB>
__device__ __forceinline__ bool is_ambiguous(float u, float margin2, float hi) {
  const float v2 = u + u;
  // boundaries 2u = n: MinMax 1 <= n <= 2K-1 (u = 0 is the argmin itself),
  // FWM and resolved n <= 2K-1 (FWM: the cut u = 0 and above; keys far in
  // the FWM tail near a negative half-integer only take the exact path).
  // Clamping 2u into [3/4, 2K - 3/4] keeps every such n and puts 2u = 0 and
  // 2u = 2K (the extrema themselves) a quarter away from any integer.
  const float c = CALIB == CAL_MINMAX ? __builtin_amdgcn_fmed3f(v2, 0.75f, hi + 0.25f)
                                      : fminf(v2, hi + 0.25f);
  return fabsf(c - rintf(c)) <= margin2;
}

// A float strictly below the boundary x (a multiple of 1/2 of either sign),
// within two ulp of it (2^-24 below x = 0).
__device__ __forceinline__ float below(float x) {
  return x - fmaxf(fabsf(x) * 0x1p-23f, 0x1p-24f);
}

template <int CALIB>
__device__ __forceinline__ void fix_ambiguous(const f32x16 &acc, const RowConst &rc,
                                           float M, float m, int K, float tau,
                                           float scale, float (&u)[16]) {
  const float Kf = (float)K, hi = 2.f * Kf - 1.f;
  uint32_t amb = 0;
#pragma unroll
  for (int r = 0; r < 16; ++r)
    amb |= (is_ambiguous<CALIB>(u[r], rc.margin2, hi) ? 1u : 0u) << r;
  while (__any(amb != 0)) {
    const int r0 = amb ? __builtin_ctz(amb) : 0;
    float x = acc[0], uu = u[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) {
      x = (r0 == r) ? acc[r] : x;
      uu = (r0 == r) ? u[r] : uu;
    }
    float rf; int up, tl;
    exact_decision(x * scale, M, m, K, CALIB, tau, rf, up, tl);
    float lo = rf + (up ? 0.5f : 0.f);
    float hv = (up && rf == Kf - 1.f) ? Kf : below(rf + (up ? 1.f : 0.5f));
    const float uf = tl ? -1.f : fminf(fmaxf(uu, lo), hv);
    if (amb) {
#pragma unroll
      for (int r = 0; r < 16; ++r) u[r] = (r0 == r) ? uf : u[r];
      amb &= amb - 1u;
    }
  }
}

// Twice the position of a key that is_ambiguous(), moved into the interval of
// its exact decision (the same values as fix_ambiguous).
template <int CALIB>
__device__ __forceinline__ float exact_v2(float s, float v, float M, float m, int K, float tau) {
  const float Kf = (float)K;
  float rf; int up, tl;
  exact_decision(s, M, m, K, CALIB, tau, rf, up, tl);
  const float lo = rf + (up ? 0.5f : 0.f);
  const float hv = (up && rf == Kf - 1.f) ? Kf : below(rf + (up ? 1.f : 0.5f));
  return 2.f * (tl ? -1.f : fminf(fmaxf(0.5f * v, lo), hv));
}

template <int CALIB>
__device__ __forceinline__ void decide_u(const f32x16 &acc, const RowConst &rc,
                                         float M, float m, int K, float tau,
                                         float scale, float (&u)[16]) {
  const float hi = 2.f * (float)K - 1.f;
  bool any = false;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    u[r] = fmaf(acc[r], rc.alpha, rc.beta);
    any |= is_ambiguous<CALIB>(u[r], rc.margin2, hi);
  }
  if (__any(any)) fix_ambiguous<CALIB>(acc, rc, M, m, K, tau, scale, u);
}

// Interval r (as float), position t, level bit and FWM tail of a key from u.
struct KeyDec {
  float rf, t;
  bool up, tail;
};
template <int CALIB>
__device__ __forceinline__ KeyDec key_of(float u, float Kf) {
  KeyDec k;
  const float fl = floorf(u);
  // MinMax: u can round a hair below 0 at the argmin; FWM keys below 0 are
  // the tail (zero weight) and the resolved grid has no lower end
  k.rf = fminf(CALIB == CAL_MINMAX ? fmaxf(fl, 0.f) : fl, Kf - 1.f);
  k.t = fminf(fmaxf(u - k.rf, 0.f), 1.f);
  k.up = k.t >= 0.5f;
  k.tail = (CALIB == CAL_FWM) && (u < 0.f);
  return k;
}

// Stored decisions in compact form. Under FWM with Nearest the backward
// needs of a key only its interval r, its level bit [t >= 1/2] and the tail
// (P^N and gamma Delta_r take no t, and FWM has no minimum channel), so the
// second pass keeps one byte per key, 1 + 2r + [t >= 1/2] for a window key
// and 0 for the tail, in the first KiB of the pair's U tile (lane l's 16
// keys at bytes 16 l + r, r the register) instead of the fp32 position u.
template <int CALIB, int RECON>
__host__ __device__ constexpr bool compact_codes() {
  return CALIB == CAL_FWM && RECON == REC_NEAREST;
}

// The lane's 16 bytes of the tile (one 16-byte store).
__device__ __forceinline__ void codes_store(float *tile, int lane, const uint32_t (&w)[4]) {
  *reinterpret_cast<uint4 *>(reinterpret_cast<char *>(tile) + 16 * lane) =
      make_uint4(w[0], w[1], w[2], w[3]);
}

__device__ __forceinline__ uint4 codes_load(const float *tile, int lane) {
  return *reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(tile) + 16 * lane);
}

// Interval, level bit and tail of register r from the lane's code words
// (t is 1 for the upper level and 0 otherwise: Nearest uses no more).
__device__ __forceinline__ KeyDec key_of_code(const uint4 &w, int r) {
  const uint32_t word = r < 4 ? w.x : (r < 8 ? w.y : (r < 12 ? w.z : w.w));
  const float cf = (float)((word >> (8 * (r & 3))) & 0xFFu);
  const float h = fmaf(cf, 0.5f, -0.5f);  // r + up / 2
  KeyDec k;
  k.rf = floorf(h);
  k.up = h - k.rf > 0.25f;
  k.t = k.up ? 1.f : 0.f;
  k.tail = cf < 0.5f;
  return k;
}

// e^{b_{r+1}} = 2^(r*hl + b1l): the raw v_exp_f32 (arguments are <= 0;
// results below the normal range flush to 0, which only drops weights
// below 1e-38 relative to the row maximum's weight 1).
__device__ __forceinline__ float grid_upper(float rf, const RowConst &rc) {
  return __builtin_amdgcn_exp2f(fmaf(rf, rc.hl, rc.b1l));
}

// ---- exponential weight functions (softmax, BF16-exp, FP8-exp) ----------
// The shift of a key from the row maximum, z = fl32(s - M) with the fp32
// score s = fl32(acc * scale): two roundings, never contracted into an fma.
__device__ __forceinline__ float score_shift(float acc, float scale, float M) {
#pragma clang fp contract(off)
  const float s = acc * scale;
  return s - M;
}

// fp32 -> bfloat16, round to nearest even, as the fp32 value with the low
// 16 bits clear (finite inputs).
__device__ __forceinline__ float bf16_rne(float x) {
  uint32_t b = __float_as_uint(x);
  b += 0x7FFFu + ((b >> 16) & 1u);
  return __uint_as_float(b & 0xFFFF0000u);
}

// a w with a zero w giving 0 whatever a is (infinite, NaN): a score gradient whose
// key has no weight. At the cost of a product: v_mul_legacy_f32, which keeps
// denormals as v_mul_f32 does. (The intrinsic and not inline asm: the compiler has
// to see the wait that an exponential's result needs before its use.)
__device__ float amdgcn_fmul_legacy(float, float) __asm("llvm.amdgcn.fmul.legacy");
__device__ __forceinline__ float mul_or_0(float a, float w) { return amdgcn_fmul_legacy(a, w); }

// Two fp32 values as one word of two bf16 (round to nearest even; a in the
// low half).
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  return (__float_as_uint(bf16_rne(a)) >> 16) | (__float_as_uint(bf16_rne(b)) & 0xFFFF0000u);
}

// Non-negative fp32 x (<= 448) -> float8_e4m3fn, round to nearest even.
// Below 2^-6 the grid is m * 2^-9 (subnormal codes m = 0..7; m = 8 is the
// smallest normal 2^-6, code 0x08); above, 3 mantissa bits with exponent
// bias 7. Returns the value; `code` receives the E4M3 byte.
__device__ __forceinline__ float e4m3_rne(float x, uint32_t &code) {
  if (x < 0x1p-6f) {
    const float m = rintf(x * 512.f);
    code = (uint32_t)m;
    return m * 0x1p-9f;
  }
  uint32_t b = __float_as_uint(x);
  b += 0x7FFFFu + ((b >> 20) & 1u);
  b &= 0xFFF00000u;
  code = (((b >> 23) - 120u) << 3) | ((b >> 20) & 7u);
  return __uint_as_float(b);
}

// Is the fp32 exponential e within the error of the fast expf() (a few
// ulp; the test window is 16 ulp) of a rounding midpoint of the target
// format? Then the rounding is decided on the correctly rounded value
// fl32(exp(x)) from the fp64 exponential instead. BF16-exp also sends
// results below the normal range there (their bf16 codes are subnormal).
template <int RECON>
__device__ __forceinline__ bool exp_near_tie(float e) {
  if constexpr (RECON == REC_BF16EXP) {
    const uint32_t lo = __float_as_uint(e) & 0xFFFFu;
    return (lo - 0x7FF0u <= 0x20u) | (e < 0x1p-126f);
  } else if constexpr (RECON == REC_FP8EXP) {
    if (e < 0x1p-6f) {
      const float y = e * 512.f;
      return fabsf(y - floorf(y) - 0.5f) <= 0x1p-16f;
    }
    const uint32_t m = __float_as_uint(e) & 0xFFFFFu;
    return m - 0x7FFF0u <= 0x20u;
  } else {
    return false;
  }
}

// Argument of the exponential: z, or bf16(z) for BF16-exp.
template <int RECON>
__device__ __forceinline__ float exp_arg(float z) {
  return RECON == REC_BF16EXP ? bf16_rne(z) : z;
}

// The fp32 exponentials e_r = fl32(exp(arg(z_r))) of the 16 keys a lane
// holds, as the weight function rounds them: fast expf(), and the fp64
// exponential for keys near a rounding midpoint (one key per lane per
// round, so the slow path runs once per round for the whole wave).
template <int RECON>
__device__ __forceinline__ void exp_tile(const float (&z)[16], float (&e)[16]) {
  uint32_t amb = 0;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    e[r] = expf(exp_arg<RECON>(z[r]));
    amb |= (exp_near_tie<RECON>(e[r]) ? 1u : 0u) << r;
  }
  if constexpr (RECON != REC_SOFTMAX) {
    while (__any(amb != 0)) {
      const int r0 = amb ? __builtin_ctz(amb) : 0;
      float x = z[0];
#pragma unroll
      for (int r = 1; r < 16; ++r) x = (r0 == r) ? z[r] : x;
      const float ex = (float)exp((double)exp_arg<RECON>(x));
      if (amb) {
#pragma unroll
        for (int r = 0; r < 16; ++r) e[r] = (r0 == r) ? ex : e[r];
        amb &= amb - 1u;
      }
    }
  }
}

// Forward weight from the stored fp32 exponential (the value U keeps for
// the backward): softmax w = e, BF16-exp w = bf16(e) (stored already
// rounded), FP8-exp w = e4m3(e).
template <int RECON>
__device__ __forceinline__ float exp_weight_of(float e) {
  if constexpr (RECON == REC_FP8EXP) {
    uint32_t c;
    return e4m3_rne(e, c);
  } else if constexpr (RECON == REC_BF16EXP) {
    return bf16_rne(e);
  } else {
    return e;
  }
}

// Workgroup barrier ordering LDS only: outstanding global stores and
// atomics are not waited for.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Work of the dQ product: query group g of qg tiles (query tiles qg g ..
// qg g + qg - 1) needs the 64-key chunks below 32 qg (g + 1) (causal) or all
// of them; cut into pieces of at most `piece` chunks (piece 0: one piece).
__host__ __device__ inline int dq_chunks(int g, int T, int causal, int qg) {
  const int all = (T + 63) / 64;
  const int need = (qg * (g + 1) + 1) / 2;
  return causal ? (need < all ? need : all) : all;
}
__host__ __device__ inline int dq_pieces(int g, int T, int causal, int piece, int qg) {
  return piece > 0 ? (dq_chunks(g, T, causal, qg) + piece - 1) / piece : 1;
}

// Tile index of the dS scratch (32x32 sub-tiles, causal: kt <= qt only).
__host__ __device__ inline size_t ds_tiles_per_slice(int nq, int causal) {
  return causal ? (size_t)nq * (nq + 1) / 2 : (size_t)nq * nq;
}
__device__ __forceinline__ size_t ds_tile(int bh, int qt, int kt, int nq,
                                          int causal) {
  const size_t in = causal ? (size_t)qt * (qt + 1) / 2 + kt : (size_t)qt * nq + kt;
  return (size_t)bh * ds_tiles_per_slice(nq, causal) + in;
}

// Element (lane l, register r) of a 32x32 fp32 tile of the scratch fields
// (dS, U) sits at (r / 4) * 256 + 4 l + r % 4: the g-th 16-byte access of
// all 64 lanes covers one contiguous KiB.
__device__ __forceinline__ void tile_load(const float *tile, int lane, float (&v)[16]) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const f32x4 x = *reinterpret_cast<const f32x4 *>(tile + 256 * g + 4 * lane);
    v[4 * g] = x[0]; v[4 * g + 1] = x[1]; v[4 * g + 2] = x[2]; v[4 * g + 3] = x[3];
  }
}
__device__ __forceinline__ void tile_store(float *tile, int lane, const float (&v)[16]) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const f32x4 x = {v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
    *reinterpret_cast<f32x4 *>(tile + 256 * g + 4 * lane) = x;
  }
}

// ---- gradient modes (the backward's `detach` argument) ---------------------
// 0 full (Eq. full), 1 detach, 2 max_only / 3 min_only (one extremum
// channel; appendix on the detached-gradient record), 4 detach with the P1
// zero-sum projection (App. B, Detach).
enum { GRAD_FULL = 0, GRAD_DETACH = 1, GRAD_MAX_ONLY = 2, GRAD_MIN_ONLY = 3, GRAD_P1 = 4 };
// the extremum channels' row sums (cM, cm) are needed
__host__ __device__ inline bool grad_channels(int g) {
  return g == GRAD_FULL || g == GRAD_MAX_ONLY || g == GRAD_MIN_ONLY;
}
__host__ __device__ inline bool grad_keep_max(int g) { return g == GRAD_FULL || g == GRAD_MAX_ONLY; }
__host__ __device__ inline bool grad_keep_min(int g) { return g == GRAD_FULL || g == GRAD_MIN_ONLY; }

// ---- bf16 inputs ---------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ float bf2f(uint32_t bits16) {
  return __uint_as_float(bits16 << 16);
}
// four consecutive inputs as fp32 (bf16 -> fp32 is exact)
__device__ __forceinline__ f32x4 load4(const float *p) {
  return *reinterpret_cast<const f32x4 *>(p);
}
__device__ __forceinline__ f32x4 load4(const uint16_t *p) {
  const uint2 x = *reinterpret_cast<const uint2 *>(p);
  const f32x4 r = {bf2f(x.x & 0xffffu), bf2f(x.x >> 16), bf2f(x.y & 0xffffu), bf2f(x.y >> 16)};
  return r;
}
__device__ __forceinline__ float load1(const float *p) { return *p; }
__device__ __forceinline__ float load1(const uint16_t *p) { return bf2f(*p); }

// v_mfma_f32_32x32x16_bf16: lane l feeds A[l%32][8(l/32) + e] and
// B[8(l/32) + e][l%32], e = 0..7; the output layout is the one of mfma32.
__device__ __forceinline__ f32x16 mfma16(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
// ---- operand pieces --------------------------------------------------------
// LDS and operand vectors that alias the element types they are staged as
typedef uint32_t u32x4 __attribute__((ext_vector_type(4), may_alias));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2), may_alias));
typedef short s16x4 __attribute__((ext_vector_type(4)));

// bf16 pieces per element: three for fp32 inputs, one for bf16 inputs.
template <typename TI> struct Pieces { static constexpr int N = sizeof(TI) == 4 ? 3 : 1; };

// The six products of two three-piece operands, smallest first.
constexpr int PROD_A[6] = {2, 1, 0, 1, 0, 0}, PROD_B[6] = {0, 1, 2, 0, 1, 0};

// Two fp32 values as one word of two bf16, round to nearest even (a low).
__device__ __forceinline__ uint32_t cvt_bf16x2(float a, float b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const bf16x2 r = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(uint32_t, r);
}

// The three pieces of eight fp32 values (exact: x = p0 + p1 + p2). What a
// piece leaves is exact in fp32, and v_dot2 (a pair of bf16 times {-1, 0} or
// {0, -1}, plus an fp32 value) takes it from the packed pair in one operation:
// seven operations for two values and their three pieces.
__device__ __forceinline__ void split8(const float (&x)[8], u32x4 (&p)[3]) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  // (kept in registers: as an inline constant -1.0 is the other half)
  uint32_t mlo = 0x0000bf80u, mhi = 0xbf800000u;
  asm("" : "+s"(mlo), "+s"(mhi));
  const bf16x2 lo = __builtin_bit_cast(bf16x2, mlo), hi = __builtin_bit_cast(bf16x2, mhi);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float a = x[2 * e], b = x[2 * e + 1];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const uint32_t w = cvt_bf16x2(a, b);
      p[i][e] = w;
      if (i < 2) {
        a = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w), lo, a, false);
        b = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w), hi, b, false);
      }
    }
  }
}
__device__ __forceinline__ bf16x8 as_op(u32x4 x) { return __builtin_bit_cast(bf16x8, x); }
// NP pieces of eight computed fp32 values: the three exact pieces, or their
// bf16 rounding
template <int NP> __device__ __forceinline__ void to_pieces(const float (&x)[8], bf16x8 (&p)[NP]) {
  if constexpr (NP == 3) {
    u32x4 w[3];
    split8(x, w);
#pragma unroll
    for (int i = 0; i < 3; ++i) p[i] = as_op(w[i]);
  } else {
    u32x4 w;
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = cvt_bf16x2(x[2 * e], x[2 * e + 1]);
    p[0] = as_op(w);
  }
}

// Operands outside the range of the pieces. Three bf16 pieces hold an fp32 value
// of 2^-100 .. 2^126, or 0, exactly, and their products stay where the value's
// do. Below, the last piece comes near bf16's smallest value; above, the first
// one rounds to infinity, and an infinity or NaN spreads to the value that it is
// split with. A product with such an operand is taken on the fp32 MFMA instead,
// with its rows read from memory. 16 operations per eight values. (The values
// themselves and not their first pieces: below 2^-134 that piece is 0.)
constexpr float PIECE_LO = 0x1p-100f, PIECE_HI = 0x1p126f;
__device__ __forceinline__ bool out_of_pieces(float x) {
  return !(fabsf(x) < PIECE_HI) | ((fabsf(x) < PIECE_LO) & (x != 0.f));
}
struct PieceCheck {
  uint32_t lo = 0xffffffffu;  // least of 2 |bits| - 1 (0: the most)
  float hi = 0.f;             // largest magnitude, NaN if there is one
  __device__ __forceinline__ void add(const float (&x)[8]) {
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      const float a = x[e], b = x[e + 1];
      lo = min(min(2u * __float_as_uint(a) - 1u, 2u * __float_as_uint(b) - 1u), lo);
      hi = __builtin_elementwise_maximum(__builtin_elementwise_maximum(fabsf(a), fabsf(b)), hi);
    }
    asm volatile("" : "+v"(lo), "+v"(hi));  // (now, or x stays live until bad())
  }
  __device__ __forceinline__ bool bad() const {
    constexpr uint32_t least = 2u * ((uint32_t)(127 - 100) << 23) - 1u;
    return (lo < least) | !(hi < PIECE_HI);
  }
};
// Score gradients are computed operands, spread over many orders of size in every
// call with wide scores, and a sum of them is as exact as its largest term: a wave's
// are out of range by the largest of all it has seen (what smaller ones then lose is
// 2^-34 of PIECE_LO each). By the largest of each lane's 16 in a tile half of the
// waves took the fp32 MFMA at a score span of 100 (q, k ~ 4 N(0,1) at d = 64,
// bwd_main 160 -> 360 us).
struct GradRange {
  float m = 0.f;  // largest magnitude, NaN if there is one
  __device__ __forceinline__ void add(const float (&x)[16]) {
#pragma unroll
    for (int r = 0; r < 16; r += 2)
      m = __builtin_elementwise_maximum(
          __builtin_elementwise_maximum(fabsf(x[r]), fabsf(x[r + 1])), m);
    asm volatile("" : "+v"(m));  // (now, or x stays live until the answer is used)
  }
  // of the whole wave
  __device__ __forceinline__ bool out() const {
    return __any(!(m < PIECE_HI)) || (__any(m > 0.f) && !__any(m >= PIECE_LO));
  }
};

// c += a b over one 16-term k-step, all its piece products.
template <int NP>
__device__ __forceinline__ f32x16 mma(const bf16x8 (&a)[NP], const bf16x8 (&b)[NP], f32x16 c) {
  if constexpr (NP == 1) return mfma16(a[0], b[0], c);
  else {
#pragma unroll
    for (int i = 0; i < 6; ++i) c = mfma16(a[PROD_A[i]], b[PROD_B[i]], c);
    return c;
  }
}

// A contraction over d (D / 16 k-steps): op(piece, s) gives an operand's
// piece `piece` at k-step s, mm(x, y, c) multiplies one of the outer and one of
// the inner operand. One piece of the outer one is live at a time; the products
// of full size come last, so that only they round at the size of the result.
template <int D, int NP, class FX, class FY, class FM>
__device__ __forceinline__ f32x16 score_tile(FX outer, FY inner, FM mm) {
  f32x16 acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
#pragma unroll
  for (int i = NP - 1; i >= 0; --i) {
    bf16x8 x[D / 16];
#pragma unroll
    for (int s = 0; s < D / 16; ++s) x[s] = outer(i, s);
#pragma unroll
    for (int j = NP - 1 - i; j >= 0; --j)
#pragma unroll
      for (int s = 0; s < D / 16; ++s) acc = mm(x[s], inner(j, s), acc);
  }
  return acc;
}
template <int D, int NP, class FA, class FB>
__device__ __forceinline__ f32x16 score_tile(FA ap, FB bp) {
  return score_tile<D, NP>(ap, bp, [](bf16x8 x, bf16x8 y, f32x16 c) { return mfma16(x, y, c); });
}
// both operands in registers
template <int D, int NP>
__device__ __forceinline__ f32x16 score_tile(const bf16x8 (&aop)[NP][D / 16],
                                             const bf16x8 (&bop)[NP][D / 16]) {
  return score_tile<D, NP>([&](int p, int s) { return aop[p][s]; },
                           [&](int p, int s) { return bop[p][s]; });
}

// The lane's operand of one 32-row tile of a [T, D] slice (rows at or beyond
// T read as zero); whether the lane holds a value out of range of the pieces.
template <int D, typename TI>
__device__ __forceinline__ bool load_rows(const TI *slice, int row, int T, int half,
                                          bf16x8 (&op)[Pieces<TI>::N][D / 16]) {
  const bool ok = row < T;
  PieceCheck check;
  const TI *src = slice + (size_t)(ok ? row : 0) * D + 8 * half;
#pragma unroll
  for (int s = 0; s < D / 16; ++s) {
    if constexpr (sizeof(TI) == 4) {
      float x[8];
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const f32x4 v = *reinterpret_cast<const f32x4 *>(src + 16 * s + 4 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e) x[4 * g + e] = ok ? v[e] : 0.f;
      }
      bf16x8 p[3];
      to_pieces<3>(x, p);
      check.add(x);
#pragma unroll
      for (int i = 0; i < 3; ++i) op[i][s] = p[i];
    } else {
      u32x4 v = *reinterpret_cast<const u32x4 *>(src + 16 * s);
      if (!ok) v = u32x4{0, 0, 0, 0};
      op[0][s] = as_op(v);
    }
  }
  return sizeof(TI) == 4 && check.bad();
}

// ---- score operands ----------------------------------------------------------
// fp32 scores stay on v_mfma_f32_32x32x2_f32, in one summation order: lane l
// feeds, at k-step s, K[key0 + l%32][(d/2) (l/32) + s] and the same of Q. An
// index decision jumps where a score's rounding does, so the order of a score's
// sum is part of the operator's result; and every fp32 value keeps all its bits
// here, whatever its size.
template <typename TI> __host__ __device__ constexpr bool fp32_scores() { return sizeof(TI) == 4; }
template <typename TI, int D> struct ScoreOp {
  bf16x8 v[1][D / 16];
  // a row of a [T, D] slice (rows at or beyond T read as zero)
  __device__ __forceinline__ void load(const TI *slice, int row, int T, int half) {
    load_rows<D>(slice, row, T, half, v);
  }
  static __device__ __forceinline__ f32x16 tile(const ScoreOp &k, const ScoreOp &q) {
    return score_tile<D, 1>(k.v, q.v);
  }
};
template <int D> struct ScoreOp<float, D> {
  float v[D / 2];
  __device__ __forceinline__ void read(const float *p) {
#pragma unroll
    for (int s = 0; s < D / 2; s += 4) {
      const f32x4 x = *reinterpret_cast<const f32x4 *>(p + s);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[s + e] = x[e];
    }
  }
  __device__ __forceinline__ void load(const float *slice, int row, int T, int half) {
    const bool ok = row < T;
    read(slice + (size_t)(ok ? row : 0) * D + half * (D / 2));
#pragma unroll
    for (int s = 0; s < D / 2; ++s) v[s] = ok ? v[s] : 0.f;
  }
  static __device__ __forceinline__ f32x16 tile(const ScoreOp &k, const ScoreOp &q) {
    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
#pragma unroll
    for (int s = 0; s < D / 2; ++s) acc = mfma32(k.v[s], q.v[s], acc);
    return acc;
  }
};

// ---- staging of row blocks in LDS ------------------------------------------
// A [ROWS, D] block staged as bf16 pieces [piece][row][D + 8] (the row stride
// of D / 2 + 4 dwords puts the 16-byte reads of eight consecutive rows in
// distinct banks). NT threads fetch eight elements each into registers
// (buffer loads: rows at or past T read as zeros) and split them when they
// are stashed.
template <int D, int ROWS, int NT, typename TI> struct Stage {
  static constexpr int NP = Pieces<TI>::N, RS = D + 8, PS = ROWS * RS, SIZE = NP * PS;
  static constexpr int V8 = ROWS * D / 8, PF = (V8 + NT - 1) / NT;
  static constexpr int RPP = NT * 8 / D;  // rows per pass
  static_assert(V8 % NT == 0 || PF == 1, "whole passes");
  u32x4 x[PF][sizeof(TI) / 2];
  __device__ __forceinline__ void fetch(const TI *src, int j0, int T, int tid) {
    const uint32_t voff = tid < V8 ? (uint32_t)tid * 8u * sizeof(TI) : 0x80000000u;
#pragma unroll
    for (int e = 0; e < PF; ++e) {
      const int rb = min(j0 + e * RPP, T);
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<TI *>(src) + (size_t)rb * D, (short)0, (T - rb) * D * (int)sizeof(TI),
          0x00020000);
#pragma unroll
      for (int g = 0; g < (int)sizeof(TI) / 2; ++g)
        x[e][g] = __builtin_bit_cast(
            u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, voff + 16u * g, 0, 0));
    }
  }
  // (check: looks the thread's values over, where given)
  __device__ __forceinline__ void stash(uint16_t *dst, int tid, PieceCheck *check = nullptr) const {
    if (V8 % NT != 0 && tid >= V8) return;
#pragma unroll
    for (int e = 0; e < PF; ++e) {
      const int idx = tid + NT * e;
      uint16_t *d = dst + (idx / (D / 8)) * RS + (idx % (D / 8)) * 8;
      if constexpr (NP == 3) {
        float f[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) f[i] = __uint_as_float(x[e][i / 4][i % 4]);
        u32x4 p[3];
        split8(f, p);
        if (check) check->add(f);
#pragma unroll
        for (int i = 0; i < 3; ++i) *reinterpret_cast<u32x4 *>(d + i * PS) = p[i];
      } else {
        *reinterpret_cast<u32x4 *>(d) = x[e][0];
      }
    }
  }
};

// A buffer resource over rows [r0, rend) of a row-major [*, D] fp32 array:
// loads at byte offsets at or past its end read as zeros (the hardware's
// range check), so ragged tails need no address clamping or masking on the
// vector units.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const float *base, int r0,
                                                          int rend, int D) {
  const int rb = min(r0, rend);
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base) + (size_t)rb * D,
                                           (short)0, (rend - rb) * D * 4, 0x00020000);
}
__device__ __forceinline__ f32x4 buffer_f32x4(__amdgpu_buffer_rsrc_t rs, uint32_t voff) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, voff, 0, 0));
}
// A [ROWS, D] fp32 block staged as it is (row stride D + 4).
template <int D, int ROWS, int NT> struct StageF32 {
  static constexpr int RS = D + 4, SIZE = ROWS * RS;  // floats
  static constexpr int V4 = ROWS * D / 4, PF = (V4 + NT - 1) / NT, RPP = NT * 4 / D;
  static_assert(V4 % NT == 0 || PF == 1, "whole passes");
  f32x4 x[PF];
  __device__ __forceinline__ void fetch(const float *src, int j0, int T, int tid) {
    const uint32_t voff = tid < V4 ? (uint32_t)tid * 16u : 0x80000000u;
#pragma unroll
    for (int e = 0; e < PF; ++e) x[e] = buffer_f32x4(row_rsrc(src, j0 + e * RPP, T, D), voff);
  }
  __device__ __forceinline__ void stash(float *dst, int tid) const {
    if (V4 % NT != 0 && tid >= V4) return;
#pragma unroll
    for (int e = 0; e < PF; ++e) {
      const int idx = tid + NT * e;
      *reinterpret_cast<f32x4 *>(dst + (idx / (D / 4)) * RS + (idx % (D / 4)) * 4) = x[e];
    }
  }
};

// Rows from r0 on of a [T, D] fp32 slice, read element by element as operands of
// the fp32 MFMA. (Rows at or past T read as zeros; d = 16: columns 16..31 are the
// next row's, in operand columns whose results nobody reads.)
template <int D> struct RowRead {
  __amdgpu_buffer_rsrc_t rs;
  uint32_t lane_off;  // bytes
  // (slice: fp32; the callers' branch for it is not taken for other types)
  template <typename TI>
  __device__ __forceinline__ RowRead(const TI *slice, int r0, int T, int lane_row, int lane_col)
      : rs(row_rsrc(reinterpret_cast<const float *>(slice), r0, T, D)),
        lane_off(4u * (uint32_t)(lane_row * D + lane_col)) {}
  __device__ __forceinline__ float at(int row, int col) const {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                         rs, lane_off + 4u * (uint32_t)(row * D + col), 0, 0));
  }
};
// (the lane's key of register r: 4 half + krel0(r))
__device__ __forceinline__ constexpr int krel0(int r) { return 8 * (r >> 2) + (r & 3); }

// Whether any thread of the workgroup's NW waves found a staged chunk out of
// range: each wave leaves its answer in flag[wave] before the barrier that
// orders the chunk's stash.
template <int NW> __device__ __forceinline__ bool any_flag(const int *flag) {
  int f = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) f |= flag[w];
  return __builtin_amdgcn_readfirstlane(f) != 0;
}

// Row-major operand: row `row` of a staged block, elements 8 half + 16 s ..
__device__ __forceinline__ bf16x8 row_op(const uint16_t *p) {
  return as_op(*reinterpret_cast<const u32x4 *>(p));
}

// Transposed operand of a staged block. ds_read_b64_tr_b16 takes, per group
// of 16 lanes, four rows of 16 columns (lane i of the group addresses row
// i / 4, columns 4 (i % 4) ..) and gives lane i the four rows' values of
// column i. The lane's column is 32 c + l % 32 and its eight k-slots are the
// rows r0 + 4 half + {0..3, 8..11}: the rows krel(8 t + e, half) with r0 =
// 16 t, that is, the lane's own registers 8 t .. 8 t + 7 of a 32x32 tile.
// tr_base() is the lane's part of the address.
template <int D, int RS = D + 8> __device__ __forceinline__ int tr_base(int lane) {
  const int col = D >= 32 ? 16 * ((lane >> 4) & 1) : 0;  // d = 16: columns 16..31 repeat, unused
  return (4 * (lane >> 5) + ((lane & 15) >> 2)) * RS + col + 4 * (lane & 3);
}
template <int RS> __device__ __forceinline__ bf16x8 tr_op(const uint16_t *p) {
  typedef s16x4 __attribute__((address_space(3))) *lds4;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)p);
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(p + 8 * RS));
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Stats view from the caller's buffer (offsets as kia_stats_offset()).
__host__ __device__ inline size_t align256(size_t x) {
  return (x + 255) & ~(size_t)255;
}

}  // namespace kia
