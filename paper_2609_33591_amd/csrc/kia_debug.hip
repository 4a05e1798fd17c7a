// kia_debug.hip -- test exports (index codes, scores), the geometry probe and
// the matrix-core peak probe.
#include "kia_device.hpp"
#include "kia_kernels.hpp"

namespace kia {

constexpr int CODES_BM = 128;
constexpr int CODES_BN = 64;

// Debug codes: the same score sub-tiles, decide_u() and key_of() as pass 2
// (REC = REC_LERP stands for both K-interval reconstructions); for an
// exponential weight function (REC >= REC_SOFTMAX) the quantized weight's
// code from the same score_shift() and exp_tile() as pass 2.
template <int D, int CALIB, int REC, typename TI>
__global__ __launch_bounds__(256) void codes_kernel(CodesArgsT<TI> a) {
  constexpr bool EXPW = is_exp_rec(REC);
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6, half = lane >> 5, l32 = lane & 31;
  const int T = a.T;
  const int nqb = (T + CODES_BM - 1) / CODES_BM;
  const int bh = blockIdx.x % a.BH;
  const int qb = nqb - 1 - (int)(blockIdx.x / a.BH);
  const int i0 = qb * CODES_BM, iw = i0 + wave * 32, row = iw + l32;
  const size_t slice = (size_t)bh * T * D;
  const float Kf = (float)a.K;
  ScoreOp<TI, D> qop;
  qop.load(a.q + slice, row < T ? row : T - 1, T, half);
  const size_t ridx = (size_t)bh * T + (row < T ? row : T - 1);
  const float Mx = a.st.M[ridx];
  const float Mn = CALIB != CAL_FWM ? a.st.m[ridx] : Mx;
  RowConst rc{};
  if constexpr (!EXPW) rc = row_const(Mx, Mn, a.K, CALIB, a.tau, a.scale);
  const int kend = a.causal ? min(T, i0 + CODES_BM) : T;
  const int ntiles = (T + CODES_BN - 1) / CODES_BN;
  for (int t = 0; t < ntiles; ++t) {
    const int j0 = t * CODES_BN;
#pragma unroll
    for (int sub = 0; sub < CODES_BN / 32; ++sub) {
      const int js = j0 + sub * 32;
      if (js >= T) continue;
      uint16_t code[16];
      if (js >= kend || (a.causal && js > iw + 31)) {
#pragma unroll
        for (int r = 0; r < 16; ++r) code[r] = 0;
      } else {
        ScoreOp<TI, D> kop;
      kop.load(a.k + slice, js + l32, T, half);
      const f32x16 acc = ScoreOp<TI, D>::tile(kop, qop);
        if constexpr (EXPW) {
          // bit 15 valid; bits 0-14 the bf16 pattern (BF16-exp) or the E4M3
          // byte (FP8-exp) of the weight, 0 for softmax (w <= 1: bit 14 clear)
          float z[16], e[16];
#pragma unroll
          for (int r = 0; r < 16; ++r) z[r] = score_shift(acc[r], a.scale, Mx);
          exp_tile<REC>(z, e);
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int j = js + krel(r, half);
            const bool valid = (j < T) & (!a.causal | (j <= row));
            uint32_t c = 0;
            if constexpr (REC == REC_BF16EXP) c = __float_as_uint(bf16_rne(e[r])) >> 16;
            if constexpr (REC == REC_FP8EXP) e4m3_rne(e[r], c);
            code[r] = valid ? (uint16_t)(0x8000u | c) : (uint16_t)0;
          }
        } else {
        float u[16];
        decide_u<CALIB>(acc, rc, Mx, Mn, a.K, a.tau, a.scale, u);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int j = js + krel(r, half);
          const bool valid = (j < T) & (!a.causal | (j <= row));
          const KeyDec kd = key_of<CALIB>(u[r], Kf);
          uint16_t c = 0;
          if (valid && CALIB == CAL_RESOLVED) {
            // bit 15 valid, bit 14 l = r + 1, bits 0-13 r (two's complement,
            // clamped to [-8192, 8191])
            const int rr = (int)fmaxf(kd.rf, -8192.f);
            c = (uint16_t)(0x8000u | (kd.up ? 0x4000u : 0u) | ((uint32_t)rr & 0x3FFFu));
          } else if (valid) {
            c = (uint16_t)(1u << 14);
            if (rc.degen) c |= (uint16_t)(1u << 15);
            else if (kd.tail) c |= (uint16_t)(1u << 13);
            else {
              const int rr = (int)kd.rf;
              const int ll = rr + (kd.up ? 1 : 0);
              c |= (uint16_t)(rr | (ll << 6));
            }
          }
          code[r] = c;
        }
        }
      }
      if (row < T) {
        uint16_t *dst = a.codes + ((size_t)bh * T + row) * T;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int j = js + krel(r, half);
          if (j < T) dst[j] = code[r];
        }
      }
    }
  }
}

// Code words of the decisions the forward stored in U (the positions u
// that pass 2 wrote and the backward reads; for an exponential weight
// function the fp32 exponential): the same format as codes_kernel, with no
// score recomputed. One wave per (b,h, 32-query tile) over all key tiles;
// codes of keys that are not valid (and of unstored tiles) are 0.
template <int CALIB, int REC>
__global__ __launch_bounds__(256) void stored_codes_kernel(StoredCodesArgs a) {
  constexpr bool EXPW = is_exp_rec(REC);
  constexpr bool COMPACT = compact_codes<CALIB, REC>();
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6, half = lane >> 5, l32 = lane & 31;
  const int T = a.T;
  const int nq = (T + 31) / 32;
  const size_t gw = (size_t)blockIdx.x * 4 + wave;
  if (gw >= (size_t)a.BH * nq) return;
  const int bh = (int)(gw / nq), qt = (int)(gw % nq);
  const int i = qt * 32 + l32;
  const float Kf = (float)a.K;
  bool degen = false;
  if (CALIB == CAL_MINMAX && i < T) {
    const size_t ridx = (size_t)bh * T + i;
    degen = (double)a.st.M[ridx] - (double)a.st.m[ridx] <= 1e-12;
  }
  for (int kt = 0; kt < nq; ++kt) {
    const bool stored = !a.causal || kt <= qt;
    float u[16];
    uint4 cw = make_uint4(0, 0, 0, 0);
    const float *tile = a.st.U + ds_tile(bh, qt, kt, nq, a.causal) * 1024;
    if (stored) {
      if constexpr (COMPACT) cw = codes_load(tile, lane);
      else tile_load(tile, lane, u);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int j = kt * 32 + krel(r, half);
      if (i >= T || j >= T) continue;
      const bool valid = stored & (!a.causal | (j <= i));
      uint32_t c = 0;
      if (valid && COMPACT) {
        const KeyDec kd = key_of_code(cw, r);
        c = 1u << 14;
        if (kd.tail) c |= 1u << 13;
        else {
          const int rr = (int)kd.rf;
          c |= (uint32_t)(rr | ((rr + (kd.up ? 1 : 0)) << 6));
        }
      } else if (valid && EXPW) {
        if constexpr (REC == REC_BF16EXP) c = __float_as_uint(bf16_rne(u[r])) >> 16;
        if constexpr (REC == REC_FP8EXP) e4m3_rne(u[r], c);
        c |= 0x8000u;
      } else if (valid) {
        const KeyDec kd = key_of<CALIB>(u[r], Kf);
        if (CALIB == CAL_RESOLVED) {
          const int rr = (int)fmaxf(kd.rf, -8192.f);
          c = 0x8000u | (kd.up ? 0x4000u : 0u) | ((uint32_t)rr & 0x3FFFu);
        } else {
          c = 1u << 14;
          if (degen) c |= 1u << 15;
          else if (kd.tail) c |= 1u << 13;
          else {
            const int rr = (int)kd.rf;
            c |= (uint32_t)(rr | ((rr + (kd.up ? 1 : 0)) << 6));
          }
        }
      }
      a.codes[((size_t)bh * T + i) * T + j] = (uint16_t)c;
    }
  }
}

// The canonical fp32 scores s = fl32(acc * scale) of every pair (the values
// the forward's extrema pass stored and every decision is taken on), 0 for
// keys that are not valid. Same sub-tile and operand loads as codes_kernel.
template <int D, typename TI>
__global__ __launch_bounds__(256) void scores_kernel(ScoresArgsT<TI> a) {
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6, half = lane >> 5, l32 = lane & 31;
  const int T = a.T;
  const int nqb = (T + CODES_BM - 1) / CODES_BM;
  const int bh = blockIdx.x % a.BH;
  const int qb = nqb - 1 - (int)(blockIdx.x / a.BH);
  const int i0 = qb * CODES_BM, iw = i0 + wave * 32, row = iw + l32;
  const size_t slice = (size_t)bh * T * D;
  ScoreOp<TI, D> qop;
  qop.load(a.q + slice, row < T ? row : T - 1, T, half);
  const int ntiles = (T + CODES_BN - 1) / CODES_BN;
  for (int t = 0; t < ntiles; ++t) {
    const int j0 = t * CODES_BN;
#pragma unroll
    for (int sub = 0; sub < CODES_BN / 32; ++sub) {
      const int js = j0 + sub * 32;
      if (js >= T) continue;
      ScoreOp<TI, D> kop;
        kop.load(a.k + slice, js + l32, T, half);
        const f32x16 acc = ScoreOp<TI, D>::tile(kop, qop);
      if (row < T) {
        float *dst = a.scores + ((size_t)bh * T + row) * T;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int j = js + krel(r, half);
          if (j < T) dst[j] = (!a.causal | (j <= row)) ? acc[r] * a.scale : 0.f;
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Geometry probe (the paper's per-row score statistics): one wave per 32
// query rows, four waves per workgroup, scores from the canonical sub-tile and decisions
// from decide_u()/key_of(), so M, the levels and the native weights are the
// forward's own. Pass A: softmax sums W_E = sum e^z and sum e^z z, the count
// of z < -6 (decided in fp64), the top-bucket mass, the bucket masses (LDS
// float atomics, [row][K + 2]: levels/intervals 0..K, the FWM tail K + 1),
// the row minimum and the LQ smallest scores of each lane (sorted insertion).
// Pass B: TV = 1/2 sum |w / W - e^z / W_E| with the forward's W.
constexpr int GEO_COUNT = 10;

template <int D, int CALIB, int RECON, int LQ>
__global__ __launch_bounds__(256) void geometry_kernel(GeoArgs a) {
  constexpr bool NEAREST = RECON == REC_NEAREST;
  __shared__ float bucket[CODES_BM * 66];  // [row][K + 2], K <= 64
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6, half = lane >> 5, l32 = lane & 31;
  const int T = a.T, K = a.K, NB = a.K + 2;
  const int nqb = (T + CODES_BM - 1) / CODES_BM;
  const int bh = blockIdx.x % a.BH;
  const int qb = nqb - 1 - (int)(blockIdx.x / a.BH);
  const int i0 = qb * CODES_BM, iw = i0 + wave * 32, row = iw + l32;
  const int lrow = wave * 32 + l32;
  const size_t slice = (size_t)bh * T * D;
  const float Kf = (float)K;
  for (int e = tid; e < CODES_BM * NB; e += 256) bucket[e] = 0.f;
  __syncthreads();
  ScoreOp<float, D> qop;
  qop.load(a.q + slice, row < T ? row : T - 1, T, half);
  float qss = 0.f, kss = 0.f;
  {
    const int rr = row < T ? row : T - 1;
    const float *src = a.q + slice + (size_t)rr * D + half * (D / 2);
    const float *ksrc = a.k + slice + (size_t)rr * D + half * (D / 2);
#pragma unroll
    for (int c = 0; c < D / 2; c += 4) {
      const f32x4 x = *reinterpret_cast<const f32x4 *>(src + c);
      const f32x4 y = *reinterpret_cast<const f32x4 *>(ksrc + c);
      qss += x[0] * x[0] + x[1] * x[1] + x[2] * x[2] + x[3] * x[3];
      kss += y[0] * y[0] + y[1] * y[1] + y[2] * y[2] + y[3] * y[3];
    }
  }
  const size_t ridx = (size_t)bh * T + (row < T ? row : T - 1);
  const float M = a.st.M[ridx];
  const float Mn = CALIB == CAL_MINMAX ? a.st.m[ridx] : M;
  const float W = a.st.W[ridx];
  const RowConst rc = row_const(M, Mn, K, CALIB, a.tau, a.scale);
  const int kend = a.causal ? min(T, i0 + CODES_BM) : T;
  const int ntiles = (kend + CODES_BN - 1) / CODES_BN;
  const int jlim = row < T ? (a.causal ? row : T - 1) : -1;

  // native weight and bucket of one key from its decided position
  auto native = [&](float u, float &w, int &b, bool &top) {
    const KeyDec kd = key_of<CALIB>(u, Kf);
    const float Eu = grid_upper(kd.rf, rc);
    const float El = Eu * rc.emh;
    const float wl = fmaf(kd.t, Eu - El, El);
    w = kd.tail ? 0.f : (NEAREST ? (kd.up ? Eu : El) : wl);
    const int lev = (int)kd.rf + (NEAREST && kd.up ? 1 : 0);
    b = kd.tail ? K + 1 : lev;
    top = !kd.tail && (NEAREST ? lev == K : (int)kd.rf == K - 1);
    if (rc.degen) { w = 1.f; b = 0; top = false; }  // App. A: weights 1, r = l = 0
  };

  float WE = 0.f, A = 0.f, topE = 0.f, smin = INFINITY, tv = 0.f;
  int cnt6 = 0;
  float low[LQ];
#pragma unroll
  for (int e = 0; e < LQ; ++e) low[e] = INFINITY;
  for (int pass = 0; pass < 2; ++pass) {
    float WEt = 0.f;
    if (pass == 1) WEt = WE;
    for (int t = 0; t < ntiles; ++t) {
      const int j0 = t * CODES_BN;
#pragma unroll
      for (int sub = 0; sub < CODES_BN / 32; ++sub) {
        const int js = j0 + sub * 32;
        if (js >= T || (a.causal && js > iw + 31)) continue;  // wave-uniform
        ScoreOp<float, D> kop;
        kop.load(a.k + slice, js + l32, T, half);
        const f32x16 acc = ScoreOp<float, D>::tile(kop, qop);
        float u[16];
        decide_u<CALIB>(acc, rc, M, Mn, K, a.tau, a.scale, u);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int j = js + krel(r, half);
          const bool valid = j <= jlim;
          const float sc = acc[r] * a.scale;
          const float z = score_shift(acc[r], a.scale, M);
          const float e = valid ? expf(z) : 0.f;
          float w; int b; bool top;
          native(u[r], w, b, top);
          if (pass == 0) {
            WE += e;
            A += e * z;
            topE += top ? e : 0.f;
            cnt6 += (valid && (double)sc - (double)M < -6.0) ? 1 : 0;
            if (valid) {
              smin = fminf(smin, sc);
              atomicAdd(&bucket[lrow * NB + b], e);
              if (sc < low[LQ - 1]) {
                float x = sc;
#pragma unroll
                for (int e2 = 0; e2 < LQ; ++e2) {
                  const float lo = fminf(low[e2], x);
                  x = fmaxf(low[e2], x);
                  low[e2] = lo;
                }
              }
            }
          } else if (valid) {
            tv += fabsf(w / W - e / WEt);
          }
        }
      }
    }
    if (pass == 0) WE += __shfl_xor(WE, 32);
  }
  A += __shfl_xor(A, 32);
  topE += __shfl_xor(topE, 32);
  cnt6 += __shfl_xor(cnt6, 32);
  smin = fminf(smin, __shfl_xor(smin, 32));
  tv += __shfl_xor(tv, 32);
  qss += __shfl_xor(qss, 32);
  kss += __shfl_xor(kss, 32);
  // the partner half's smallest scores merged into this lane's list (read
  // in full first: both halves merge at once)
  float other[LQ];
#pragma unroll
  for (int e = 0; e < LQ; ++e) other[e] = __shfl_xor(low[e], 32);
#pragma unroll
  for (int e = 0; e < LQ; ++e) {
    float x = other[e];
#pragma unroll
    for (int e2 = 0; e2 < LQ; ++e2) {
      const float lo = fminf(low[e2], x);
      x = fmaxf(low[e2], x);
      low[e2] = lo;
    }
  }
  __syncthreads();
  if (half == 1 || row >= T) return;
  const int n = a.causal ? row + 1 : T;
  float Hq = 0.f;
  for (int b = 0; b < NB; ++b) {
    const float mb = bucket[lrow * NB + b];
    Hq += mb > 0.f ? mb * logf(mb) : 0.f;
  }
  const float lWE = logf(WE);
  // 0.1% quantile of z: linear interpolation at (n - 1) * 0.001 between
  // the order statistics lo and lo + 1 of the row's scores
  const double pos = (double)(n - 1) * 0.001;
  const int lo = (int)floor(pos), hi = lo + 1 < n ? lo + 1 : lo;
  float slo = low[0], shi = low[0];
#pragma unroll
  for (int e = 1; e < LQ; ++e) {
    slo = e == lo ? low[e] : slo;
    shi = e == hi ? low[e] : shi;
  }
  const double zlo = (double)slo - (double)M, zhi = (double)shi - (double)M;
  float *o = a.out + ((size_t)bh * T + row) * GEO_COUNT;
  const float span = M - smin;
  o[0] = span;
  o[1] = CALIB == CAL_MINMAX ? span / Kf : a.tau / Kf;
  o[2] = (float)(zlo + (pos - (double)lo) * (zhi - zlo));
  o[3] = sqrtf(qss);
  o[4] = sqrtf(kss);
  o[5] = lWE - A / WE;
  o[6] = (float)cnt6 / (float)n;
  o[7] = topE / WE;
  o[8] = expf(lWE - Hq / WE);
  o[9] = 0.5f * tv;
}

#define KIA_GEO_INST(D)                                                        \
  template __global__ void geometry_kernel<D, CAL_MINMAX, REC_LERP, 3>(GeoArgs);     \
  template __global__ void geometry_kernel<D, CAL_MINMAX, REC_NEAREST, 3>(GeoArgs);  \
  template __global__ void geometry_kernel<D, CAL_FWM, REC_LERP, 3>(GeoArgs);        \
  template __global__ void geometry_kernel<D, CAL_FWM, REC_NEAREST, 3>(GeoArgs);     \
  template __global__ void geometry_kernel<D, CAL_MINMAX, REC_LERP, 12>(GeoArgs);    \
  template __global__ void geometry_kernel<D, CAL_MINMAX, REC_NEAREST, 12>(GeoArgs); \
  template __global__ void geometry_kernel<D, CAL_FWM, REC_LERP, 12>(GeoArgs);       \
  template __global__ void geometry_kernel<D, CAL_FWM, REC_NEAREST, 12>(GeoArgs);    \
  template __global__ void geometry_kernel<D, CAL_MINMAX, REC_LERP, 67>(GeoArgs);    \
  template __global__ void geometry_kernel<D, CAL_MINMAX, REC_NEAREST, 67>(GeoArgs); \
  template __global__ void geometry_kernel<D, CAL_FWM, REC_LERP, 67>(GeoArgs);       \
  template __global__ void geometry_kernel<D, CAL_FWM, REC_NEAREST, 67>(GeoArgs);
KIA_GEO_INST(16)
KIA_GEO_INST(32)
KIA_GEO_INST(64)
KIA_GEO_INST(128)

// ---------------------------------------------------------------------------
// Matrix-core peak probe (a measurement aid, not part of the operator): four
// independent accumulator chains of v_mfma_f32_32x32x2_f32 on register
// operands, `iters` rounds per wave. Workgroup 0's first wave records the
// shader clock counter and the 100 MHz constant-rate counter around its loop.
__global__ __launch_bounds__(256) void mfma_probe_kernel(unsigned long long *out, int iters) {
  const int lane = threadIdx.x & 63;
  const float x = 0.001f * (float)lane, y = 1.f - 0.0005f * (float)lane;
  f32x16 c0, c1, c2, c3;
#pragma unroll
  for (int e = 0; e < 16; ++e) c0[e] = c1[e] = c2[e] = c3[e] = 0.f;
  __builtin_amdgcn_sched_barrier(0);
  const unsigned long long t0 = __builtin_amdgcn_s_memtime();
  const unsigned long long r0 = __builtin_amdgcn_s_memrealtime();
  __builtin_amdgcn_sched_barrier(0);
  for (int i = 0; i < iters; ++i) {
    c0 = mfma32(x, y, c0);
    c1 = mfma32(y, x, c1);
    c2 = mfma32(x, x, c2);
    c3 = mfma32(y, y, c3);
  }
  __builtin_amdgcn_sched_barrier(0);
  float sum = 0.f;
#pragma unroll
  for (int e = 0; e < 16; ++e) sum += c0[e] + c1[e] + c2[e] + c3[e];
  const unsigned long long t1 = __builtin_amdgcn_s_memtime();
  const unsigned long long r1 = __builtin_amdgcn_s_memrealtime();
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    out[0] = t0; out[1] = t1; out[2] = r0; out[3] = r1;
  }
  if (sum == -1.f) out[0] = 0;  // never true (all products are >= 0): keeps the chains live
}

#define KIA_CODES_INST(D)                                                               \
  template __global__ void codes_kernel<D, CAL_MINMAX, REC_LERP, float>(CodesArgs);     \
  template __global__ void codes_kernel<D, CAL_FWM, REC_LERP, float>(CodesArgs);        \
  template __global__ void codes_kernel<D, CAL_RESOLVED, REC_LERP, float>(CodesArgs);   \
  template __global__ void codes_kernel<D, CAL_FWM, REC_SOFTMAX, float>(CodesArgs);     \
  template __global__ void codes_kernel<D, CAL_FWM, REC_BF16EXP, float>(CodesArgs);     \
  template __global__ void codes_kernel<D, CAL_FWM, REC_FP8EXP, float>(CodesArgs);      \
  template __global__ void codes_kernel<D, CAL_MINMAX, REC_LERP, uint16_t>(CodesArgs16);\
  template __global__ void codes_kernel<D, CAL_FWM, REC_LERP, uint16_t>(CodesArgs16);   \
  template __global__ void codes_kernel<D, CAL_RESOLVED, REC_LERP, uint16_t>(CodesArgs16);
KIA_CODES_INST(16)
KIA_CODES_INST(32)
KIA_CODES_INST(64)
KIA_CODES_INST(128)
template __global__ void stored_codes_kernel<CAL_MINMAX, REC_LERP>(StoredCodesArgs);
template __global__ void stored_codes_kernel<CAL_FWM, REC_LERP>(StoredCodesArgs);
template __global__ void stored_codes_kernel<CAL_FWM, REC_NEAREST>(StoredCodesArgs);
template __global__ void stored_codes_kernel<CAL_RESOLVED, REC_LERP>(StoredCodesArgs);
template __global__ void stored_codes_kernel<CAL_FWM, REC_SOFTMAX>(StoredCodesArgs);
template __global__ void stored_codes_kernel<CAL_FWM, REC_BF16EXP>(StoredCodesArgs);
template __global__ void stored_codes_kernel<CAL_FWM, REC_FP8EXP>(StoredCodesArgs);
#define KIA_SCORES_INST(D)                                                  \
  template __global__ void scores_kernel<D, float>(ScoresArgsT<float>);     \
  template __global__ void scores_kernel<D, uint16_t>(ScoresArgsT<uint16_t>);
KIA_SCORES_INST(16)
KIA_SCORES_INST(32)
KIA_SCORES_INST(64)
KIA_SCORES_INST(128)

}  // namespace kia
