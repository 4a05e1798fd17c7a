// kia_kernels.hpp -- argument blocks and kernel declarations shared between
// the host entry points (kia_abi.hip) and the kernel sources.
#pragma once

#include "kia_device.hpp"

namespace kia {

// TI: element type of the inputs q, k, v, dO (float, or uint16_t holding
// bf16 bits); outputs and statistics are fp32 either way.
template <typename TI> struct FwdArgsT {
  const TI *q, *k, *v;
  float *o;
  Stats st;
  int BH, T, K, calib, recon, causal;
  float tau, scale;
  uint16_t *o16 = nullptr;  // bf16-output variant: O as bf16 here instead of o
  int keep = 1;  // 0 (forward only): pass 2 stores no decisions in U
  // grid constants that do not depend on the row (FWM and resolved; see
  // fwd_row_const): K / tau, and as RowConst alpha, hl, b1l, emh
  double gc = 0.0;
  float ga = 0.f, ghl = 0.f, gb1l = 0.f, gemh = 1.f;
};

// Launch shape of the forward: NBUF staging buffers per tensor, OCC waves per
// SIMD (one where a chunk or the key parts' sums take more than half the LDS; fp32
// inputs at d = 128 with O_l: one as well, two spill. Without O_l two are faster,
// MinMax Nearest B1 H40 T1024 159 -> 126 us). fp32 scores come from the fp32
// MFMA (EX) and K is staged as it is. KEEP: the scores are kept in U between the
// passes, and V takes K's place in LDS in the second. Computing them again
// instead grows with d, the trip through U does not, and small grids have the
// bandwidth to spare. Measured (us, kept / again), B8 H12 T1024 (4 x 1), MinMax
// LERP: d = 16 117 / 99, d = 32 145 / 130, d = 64 175 / 213; B1 H12 T1024 (1 x 4),
// FWM Nearest Prob-STE: d = 16 27.3 / 28.3, d = 32 31.8 / 34.7.
template <typename TI, int D, int RECON, bool OL, int RG, int KP> struct FwdShape {
  static constexpr bool EX = fp32_scores<TI>();
  static constexpr bool KEEP = EX && (D >= 64 || RG < 4);
  // bytes of one staged block of V and of K
  static constexpr int VB = Pieces<TI>::N * 32 * KP * (D + 8) * 2;
  static constexpr int KB = EX ? 32 * KP * (D + 4) * 4 : VB;
  static constexpr int WGS = RG * KP == 8 ? 1 : 2;  // workgroups that make two waves per SIMD
  static constexpr int LDS = RG == 1 || KEEP ? VB : VB + KB;  // a buffer for each tensor, or one for both
  // values a lane of key part > 0 hands to part 0 at the end, and their bytes
  static constexpr int NRED = (D >= 32 ? D / 32 : 1) * 16 * (OL ? 2 : 1) + 2;
  static constexpr int RED = (KP - 1) * RG * 64 * NRED * 4;
  static constexpr int OCC =
      (LDS > RED ? LDS : RED) * WGS > 156 * 1024 || (EX && D == 128 && OL) ? 1 : 2;
  static constexpr int NBUF =
      2 * (KEEP ? VB : VB + KB) * (OCC == 2 ? WGS : 1) <= 156 * 1024 ? 2 : 1;
};

// Row constants of the forward: as row_const(), with what FWM and the
// resolved grid share across rows taken from the arguments.
template <int CALIB, typename TI>
__device__ __forceinline__ RowConst fwd_row_const(float M, float m, const FwdArgsT<TI> &a) {
  if constexpr (CALIB == CAL_MINMAX) {
    return row_const(M, m, a.K, CALIB, a.tau, a.scale);
  } else {
    RowConst rc{};
    const double Kd = (double)a.K, t = (double)a.tau;
    rc.alpha = a.ga; rc.hl = a.ghl; rc.b1l = a.gb1l; rc.emh = a.gemh;
    rc.beta = (float)(Kd - (double)M * a.gc);
    const double A = CALIB == CAL_RESOLVED
                         ? fmax(fabs((double)M), fabs((double)m)) + t + ((double)M - (double)m)
                         : fabs((double)M) + t;
    rc.margin2 = (float)ldexp(3.0 * a.gc * A + 2.0 * Kd, -20);
    return rc;
  }
}

template <typename TI> struct CodesArgsT {
  const TI *q, *k;
  Stats st;
  uint16_t *codes;
  int BH, T, K, calib, causal;
  float tau, scale;
};

template <typename TI> struct BwdArgsT {
  const TI *q, *k, *v;
  const float *o;
  const TI *dO;
  float *dq, *dk, *dv;
  Stats st;
  int BH, T, K, calib, recon, ste, grad, causal;  // grad: GRAD_* mode
  // qsplit > 1: each key block's query range is split over qsplit workgroups
  // of bwd_main, which add their dK/dV into dk/dv (zeroed by bwd_pre)
  int qsplit;
  // dq_piece > 0: bwd_dq cuts each query group's 64-key chunks into pieces
  // of at most dq_piece chunks, which add into dq (zeroed by bwd_pre)
  int dq_piece;
  // 1 (qsplit 3 or 4, dq_piece 0): the third and fourth part add their dV into dq,
  // which bwd_dq adds to dv before it writes dq. A sum of two does not depend on
  // their order, so that dV is the same on every call.
  int fold = 0;
  // 1: every reduction in a fixed order (kia_set_deterministic): row sums
  // through st.part, calibration terms gathered per key, ties one wave per
  // slice; qsplit = 1 and dq_piece = 0
  int det = 0;
  float tau, scale;
  // bf16-output variant: the forward's O read as bf16 from o16 (instead of
  // o) and dV written as bf16 to dv16 (instead of dv); dq and dk then point
  // at the fp32 accumulators in stats, which cast_bf16_kernel rounds at the end
  const uint16_t *o16 = nullptr;
  uint16_t *dv16 = nullptr;
  float ghl = 0.f, gemh = 1.f;  // grid constants of FWM and resolved (as RowConst hl, emh)
};

// Waves per SIMD of the backward's main kernel: at d = 128 the three pieces of
// V and the dV and dK accumulators take more than half the registers.
template <typename TI, int D> struct MainShape {
  static constexpr int OCC = sizeof(TI) == 4 && D == 128 ? 1 : 2;
};

// Waves per SIMD of the dQ kernel. (fp32 at d = 64: in 128 registers the q rows
// that are loaded ahead of the key loop spill, and the loop waits for them. B8 H12
// T1024, four / three waves: 104 / 78.5 us.)
template <typename TI, int D> struct DqShape {
  static constexpr int OCC = D == 128 ? (sizeof(TI) == 4 ? 2 : 3) : (sizeof(TI) == 4 && D == 64 ? 3 : 4);
};

using FwdArgs = FwdArgsT<float>;
using CodesArgs = CodesArgsT<float>;
using BwdArgs = BwdArgsT<float>;
using FwdArgs16 = FwdArgsT<uint16_t>;
using CodesArgs16 = CodesArgsT<uint16_t>;
using BwdArgs16 = BwdArgsT<uint16_t>;

template <typename TI, int D, int CALIB, int RECON, bool OL, int RG, int KP>
__global__ void fwd_kernel(FwdArgsT<TI> a);
template <int D, int CALIB, int REC, typename TI> __global__ void codes_kernel(CodesArgsT<TI> a);
// test exports: the code words of the decisions stored in U (no score
// recomputation), and the canonical fp32 score sub-tiles
struct StoredCodesArgs {
  Stats st;
  uint16_t *codes;
  int BH, T, K, causal;
};
template <int CALIB, int REC> __global__ void stored_codes_kernel(StoredCodesArgs a);
template <typename TI> struct ScoresArgsT {
  const TI *q, *k;
  float *scores;
  int BH, T, causal;
  float scale;
};
template <int D, typename TI> __global__ void scores_kernel(ScoresArgsT<TI> a);
template <int D, typename TI> __global__ void bwd_pre_kernel(BwdArgsT<TI> a);
template <typename TI, int D, int CALIB, int RECON>
__global__ void bwd_main_kernel(BwdArgsT<TI> a);
// query tiles per bwd_dq workgroup (x 2 key halves = its waves): two for
// d <= 64 (smaller workgroups, four per CU, balance the causal groups
// better), four for d = 128 (where the larger K chunk per thread would cost)
constexpr int dq_tiles(int d) { return d <= 64 ? 2 : 4; }
template <typename TI, int D, int QG> __global__ void bwd_dq_kernel(BwdArgsT<TI> a);
template <int D, typename TI> __global__ void bwd_ties_kernel(BwdArgsT<TI> a);
template <int D, typename TI> __global__ void bwd_p1_kernel(BwdArgsT<TI> a);
// deterministic backward: row sums from the key blocks' partials; the
// calibration terms of rows with unique extrema gathered onto dK per key
template <typename TI> __global__ void row_sums_kernel(BwdArgsT<TI> a);
template <int D, typename TI, int NW> __global__ void calib_gather_kernel(BwdArgsT<TI> a);
__global__ void cast_bf16_kernel(const float *src, uint16_t *dq, uint16_t *dk, uint16_t *dv,
                                 size_t n8);
struct GradArgs {
  Stats st;
  float *g_self, *cM, *cm;
  int BH, T, calib, causal, bf16;
};
__global__ void score_grad_kernel(GradArgs a);
struct GeoArgs {
  const float *q, *k;
  Stats st;
  float *out;  // [BH, T, 10]
  int BH, T, K, causal;
  float tau, scale;
};
template <int D, int CALIB, int RECON, int LQ> __global__ void geometry_kernel(GeoArgs a);
__global__ void mfma_probe_kernel(unsigned long long *out, int iters);

}  // namespace kia
