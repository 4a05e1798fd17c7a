// kia_bf16.hip -- the bf16-input variant of the forward and backward on
// gfx950: q, k, v and dO are bf16, every product runs on the bf16 MFMA
// (v_mfma_f32_32x32x16_bf16) with fp32 accumulation, and everything else
// (scores, extrema, index decisions, weights, normalizers, gradients of the
// scores, outputs) is fp32 as in the fp32 path. The computed operands of
// the second products (weights, dS) are rounded to bf16 for the MFMA.
//
// The kernels mirror the fp32 ones (kia_fwd.hip, kia_bwd.hip): same
// workgroup shapes and stats fields (the forward stores the score tiles in
// U and replaces them by the decided positions u, which the backward reads;
// recomputing the scores in the second pass is cheap on the bf16 MFMA but
// its extra staging registers cost more than the tile traffic at d = 128).
// The dS scratch holds bf16 (2 KiB per tile), the dQ product's operand
// precision. They also differ in the operand staging. A 32x32x16 MFMA takes 8 consecutive k-slots per lane
// half; in the products whose k index is a key (P V, dS K), a lane's own
// weight (or dS) registers r = 8t .. 8t+7 are the k-slots, that is the keys
// krel(8t + e, h), so V and K are staged transposed in LDS and a lane reads
// its 8 operands as two 8-byte runs of 4 consecutive keys. In the products
// whose k index is a query (P^T dO, dS^T Q), P and dS go through the
// wave-private transpose of the fp32 path and dO, Q are staged transposed.
#include <type_traits>

#include "kia_device.hpp"
#include "kia_kernels.hpp"

namespace kia {

constexpr int H16_CH = 64;  // keys per streamed chunk
constexpr int H16_TS = 68;  // row stride (bf16) of a transposed 64-key chunk
constexpr int H16_QT = 40;  // row stride (bf16) of a transposed 32-query tile
constexpr int H16_XS = 40;  // wave-private transpose row stride (bf16)
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));

template <int D> struct Dims16 {
  static constexpr int NC = D >= 32 ? D / 32 : 1;  // 32-column output blocks
  static constexpr int RS = D + 8;                  // row-major LDS row (bf16)
};

__device__ __forceinline__ bf16x8 pair_bf16x8(uint2 lo, uint2 hi) {
  return as_bf16x8(make_uint4(lo.x, lo.y, hi.x, hi.y));
}

// Register prefetch of a [ROWS, D] bf16 slice by NT threads in blocks of 4
// rows x 8 columns (one 16-byte load per row). The loads are unconditional
// (clamped rows) and masked when stashed into LDS, row-major or transposed.
template <int D, int ROWS, int NT> struct Blocks16 {
  static constexpr int CB = D / 8;
  static constexpr int NB = (ROWS / 4) * CB;
  static constexpr int PB = (NB + NT - 1) / NT;
  uint4 x[PB][4];
  uint32_t ok;
  __device__ __forceinline__ void fetch(const uint16_t *slice, int j0, int T, int tid) {
    ok = 0;
#pragma unroll
    for (int e = 0; e < PB; ++e) {
      const int b = tid + NT * e;
      const bool bv = b < NB;
      const int rb = bv ? b / CB : 0, cb = bv ? b % CB : 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = j0 + 4 * rb + i;
        const bool v = bv & (row < T);
        ok |= (v ? 1u : 0u) << (4 * e + i);
        x[e][i] = *reinterpret_cast<const uint4 *>(slice + (size_t)(v ? row : 0) * D + 8 * cb);
      }
    }
  }
  template <int RSTRIDE>
  __device__ __forceinline__ void stash_rows(uint16_t *dst, int tid) const {
#pragma unroll
    for (int e = 0; e < PB; ++e) {
      const int b = tid + NT * e;
      if (b < NB) {
        const int rb = b / CB, cb = b % CB;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          *reinterpret_cast<uint4 *>(dst + (4 * rb + i) * RSTRIDE + 8 * cb) =
              ((ok >> (4 * e + i)) & 1u) ? x[e][i] : make_uint4(0, 0, 0, 0);
      }
    }
  }
  // column 8cb + c of the block's 4 rows -> dst[(8cb + c) * TSTRIDE + 4rb ..]
  template <int TSTRIDE>
  __device__ __forceinline__ void stash_cols(uint16_t *dst, int tid) const {
#pragma unroll
    for (int e = 0; e < PB; ++e) {
      const int b = tid + NT * e;
      if (b < NB) {
        const int rb = b / CB, cb = b % CB;
        uint32_t w[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint4 v = ((ok >> (4 * e + i)) & 1u) ? x[e][i] : make_uint4(0, 0, 0, 0);
          w[i][0] = v.x; w[i][1] = v.y; w[i][2] = v.z; w[i][3] = v.w;
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          const int dw = c >> 1;
          uint32_t p01, p23;
          if (c & 1) {
            p01 = (w[0][dw] >> 16) | (w[1][dw] & 0xffff0000u);
            p23 = (w[2][dw] >> 16) | (w[3][dw] & 0xffff0000u);
          } else {
            p01 = (w[0][dw] & 0xffffu) | (w[1][dw] << 16);
            p23 = (w[2][dw] & 0xffffu) | (w[3][dw] << 16);
          }
          *reinterpret_cast<uint2 *>(dst + (8 * cb + c) * TSTRIDE + 4 * rb) = make_uint2(p01, p23);
        }
      }
    }
  }
};

// ---------------------------------------------------------------------------
// dQ (bf16 inputs) = scale * (dS K + calibration terms): as bwd_dq_kernel,
// with each 64-key chunk of K staged transposed in bf16 and the fp32 dS
// tiles (stored in bf16 by bwd16_main_kernel) as the A operand.
template <int D>
__global__ __launch_bounds__(512) void bwd16_dq_kernel(BwdArgs16 a) {
  constexpr int NC = Dims16<D>::NC;
  constexpr int KT = D * H16_TS;  // bf16 per transposed chunk
  constexpr int STAGE_B = 2 * KT * 2;
  constexpr int RED_B = 4 * NC * 16 * 64 * 4;
  constexpr int SMB = STAGE_B > RED_B ? STAGE_B : RED_B;
  __shared__ __attribute__((aligned(16))) unsigned char smem[SMB];
  uint16_t *Kt = reinterpret_cast<uint16_t *>(smem);

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6, half = lane >> 5, l32 = lane & 31;
  const int pq = wave & 3, kh = wave >> 2;
  const int T = a.T;
  const int nq = (T + 31) / 32;
  const int npq = (nq + 3) / 4;
  const int bh = blockIdx.x % a.BH;
  const int g = npq - 1 - (int)(blockIdx.x / a.BH);
  const int qt = 4 * g + pq;
  const bool live = qt < nq;
  const int qtc = live ? qt : nq - 1;
  const size_t slice = (size_t)bh * T * D;
  const uint16_t *ks = a.k + slice;
  const int kend = a.causal ? min(T, (4 * g + 4) * 32) : T;
  const int nstep = (kend + 63) / 64;
  const int ktmine = a.causal ? qtc : nq - 1;
  const int npw = !live || ktmine < kh ? 0 : min(nstep, (ktmine - kh) / 2 + 1);
  const bool minmax = a.calib == CAL_MINMAX;

  f32x16 acc[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[c][e] = 0.f;

  Blocks16<D, 64, 512> kA, kB;
  uint4 dA[2], dB[2];
  auto fetch = [&](int p, Blocks16<D, 64, 512> &kx, uint4 (&dx)[2]) {
    kx.fetch(ks, p * 64, T, tid);
    const int kt = min(2 * p + kh, ktmine);
    // the bf16 dS tile of bwd16_main_kernel
    const uint16_t *src = reinterpret_cast<const uint16_t *>(a.st.dS) +
                          ds_tile(bh, qtc, kt, nq, a.causal) * 1024 + 8 * lane;
#pragma unroll
    for (int t = 0; t < 2; ++t) dx[t] = *reinterpret_cast<const uint4 *>(src + 512 * t);
  };
  auto mma = [&](int buf, const uint4 (&dx)[2]) {
    const uint16_t *kb = Kt + buf * KT + kh * 32 + 4 * half;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const bf16x8 av = as_bf16x8(dx[t]);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int col = 32 * c + l32;
        const uint16_t *kr = kb + (col < D ? col : 0) * H16_TS + 16 * t;
        uint2 lo = *reinterpret_cast<const uint2 *>(kr);
        uint2 hi = *reinterpret_cast<const uint2 *>(kr + 8);
        if (col >= D) { lo = make_uint2(0, 0); hi = lo; }
        acc[c] = mfma16(av, pair_bf16x8(lo, hi), acc[c]);
      }
    }
  };
  fetch(0, kA, dA);
  kA.template stash_cols<H16_TS>(Kt, tid);
  fetch(min(1, nstep - 1), kB, dB);
  lds_barrier();
  for (int p = 0; p < nstep; p += 2) {
    if (p < npw) mma(0, dA);
    kB.template stash_cols<H16_TS>(Kt + KT, tid);
    fetch(min(p + 2, nstep - 1), kA, dA);
    lds_barrier();
    if (p + 1 >= nstep) break;
    if (p + 1 < npw) mma(1, dB);
    kA.template stash_cols<H16_TS>(Kt, tid);
    fetch(min(p + 3, nstep - 1), kB, dB);
    lds_barrier();
  }
  {
    float *red = reinterpret_cast<float *>(smem) + pq * (NC * 16 * 64) + lane;
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
  const int row = qt * 32 + l32;
  const size_t ridx = (size_t)bh * T + (row < T ? row : T - 1);
  bool ok = false;
  float cMt = 0.f, cm = 0.f;
  int am = 0, an = 0;
  if (grad_channels(a.grad) && row < T && a.st.rowrec[ridx * RR_COUNT + RR_FLAGS] == 0.f) {
    const int nmax = a.st.nmax[ridx];
    const int nmin = minmax ? a.st.nmin[ridx] : 1;
    ok = (nmax == 1) & (nmin == 1);
    const float ss = a.st.sself[ridx];
    cMt = minmax ? a.st.cM[ridx] : -ss;
    cm = minmax ? -(ss + cMt) : 0.f;
    if (!grad_keep_max(a.grad)) cMt = 0.f;
    if (!grad_keep_min(a.grad)) cm = 0.f;
    am = a.st.amax[ridx];
    an = minmax ? a.st.amin[ridx] : am;
  }
  if (!ok) { cMt = 0.f; cm = 0.f; am = 0; an = 0; }
  if (kh == 0) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int src = krel(e, half);
      const float fM = __shfl(cMt, src), fm = __shfl(cm, src);
      const int iam = __shfl(am, src), ian = __shfl(an, src);
      const int qrow = qt * 32 + src;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int n = 32 * c + l32;
        const int nn = n < D ? n : 0;
        float v = acc[c][e];
        v = fmaf(fM, load1(ks + (size_t)iam * D + nn), v);
        v = fmaf(fm, load1(ks + (size_t)ian * D + nn), v);
        if (qrow < T && n < D) a.dq[slice + (size_t)qrow * D + n] = a.scale * v;
      }
    }
  }
  // scatter onto the argmax/argmin keys of dK (the deterministic backward
  // gathers these per key instead: one record per row for it)
  if (a.det && grad_channels(a.grad) && kh == 0 && half == 0 && row < T)
    put_calib_record(a.st.part, ridx, ok, minmax, am, an, cMt * a.scale, cm * a.scale);
  if (grad_channels(a.grad) && !a.det) {
    constexpr int NE = (D + 63) / 64;
    for (int rr0 = 16 * kh; rr0 < 16 * kh + 16; rr0 += 8) {
      float qv[8][NE];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int qrow = qt * 32 + rr0 + u;
#pragma unroll
        for (int x = 0; x < NE; ++x) {
          const int n = lane + 64 * x;
          const int qr = qrow < T ? qrow : T - 1, nn = n < D ? n : 0;
          qv[u][x] = load1(a.q + slice + (size_t)qr * D + nn);
        }
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int rr = rr0 + u;
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
}

#define KIA_B16_INST(D)                                                                  \
  template __global__ void bwd16_dq_kernel<D>(BwdArgs16);
KIA_B16_INST(16)
KIA_B16_INST(32)
KIA_B16_INST(64)
KIA_B16_INST(128)

}  // namespace kia
