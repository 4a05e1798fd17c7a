// kia_abi.hip -- extern "C" entry points of libkia (declared in include/kia.h).
// Host side only: argument validation (before any launch), the stats layout,
// kernel selection by head dimension, and launches on the caller's stream.
#include <math.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <vector>

#include "kia.h"
#include "kia_kernels.hpp"

namespace {

using namespace kia;

constexpr int NFIELD = 16;  // KIA_STAT_ACC last (size 0 unless the bf16-output layout)

bool need_ol(int recon, int ste) {
  return recon == KIA_RECON_NEAREST && ste == KIA_STE_PROB;
}

// Byte size of each stats field (KIA_STAT_* order).
size_t field_bytes(int B, int H, int T, int d, int recon, int ste, int causal,
                   int field) {
  const size_t R = (size_t)B * H * T;
  switch (field) {
    case KIA_STAT_ROWREC: return R * RR_COUNT * sizeof(float);
    // present for every operator, so that no field's offset depends on
    // recon or ste (only Nearest with Prob-STE writes it)
    case KIA_STAT_OL: return R * (size_t)d * sizeof(float);
    case KIA_STAT_DS:
    case KIA_STAT_U:
      return (size_t)B * H * ds_tiles_per_slice((T + 31) / 32, causal) * 1024 * sizeof(float);
    // (also the calibration records of the deterministic gather: 4 per row)
    case KIA_STAT_PART:
      return std::max<size_t>(2 * (size_t)((T + 127) / 128), 4) * R * sizeof(float);
    case KIA_STAT_ACC: return 0;  // only in kia_stats_bytes_bf16o
    default: return R * 4;
  }
}

size_t field_offset(int B, int H, int T, int d, int recon, int ste, int causal,
                    int field) {
  size_t off = 0;
  for (int f = 0; f < field; ++f)
    off += align256(field_bytes(B, H, T, d, recon, ste, causal, f));
  return off;
}

int check_shape(int B, int H, int T, int d) {
  if (B < 1 || H < 1 || T < 1 || T > 65536) return KIA_ERR_SHAPE;
  if (d != 16 && d != 32 && d != 64 && d != 128) return KIA_ERR_HEADDIM;
  const long double n = (long double)B * H * T * d;
  if (n >= 2147483648.0L) return KIA_ERR_SHAPE;
  return KIA_OK;
}

bool recon_ok(int recon) { return recon >= KIA_RECON_LERP && recon <= KIA_RECON_FP8EXP; }

// The statistics (bf16-output accumulators included) must fit in
// KIA_MAX_STATS_BYTES: the two tile fields grow as T^2.
int check_size(int B, int H, int T, int d, int causal) {
  const size_t bytes = field_offset(B, H, T, d, 0, 0, causal, NFIELD) +
                       align256((size_t)3 * B * H * T * d * sizeof(float));
  return bytes > (size_t)KIA_MAX_STATS_BYTES ? KIA_ERR_SHAPE : KIA_OK;
}

int check_args(int B, int H, int T, int d, int K, int calib, float tau,
               int recon, int ste, int detach, int causal) {
  int rc = check_shape(B, H, T, d);
  if (rc) return rc;
  if (is_exp_rec(recon)) {
    // exponential weight functions: K, calib, tau and ste are not used
    if (!recon_ok(recon) || detach < GRAD_FULL || detach > KIA_GRAD_NONE ||
        (causal != 0 && causal != 1))
      return KIA_ERR_ENUM;
    return check_size(B, H, T, d, causal);
  }
  if (K < 1 || K > 64) return KIA_ERR_K;
  if (calib < KIA_CALIB_MINMAX || calib > KIA_CALIB_RESOLVED || (recon != 0 && recon != 1) ||
      (ste != 0 && ste != 1) || detach < GRAD_FULL || detach > KIA_GRAD_NONE ||
      (causal != 0 && causal != 1))
    return KIA_ERR_ENUM;
  if (calib != KIA_CALIB_MINMAX && !(tau > 0.f && isfinite(tau))) return KIA_ERR_TAU;
  return check_size(B, H, T, d, causal);
}

bool al16(const void *p) { return ((uintptr_t)p & 15u) == 0; }
bool al256(const void *p) { return ((uintptr_t)p & 255u) == 0; }

Stats make_stats(void *base, int B, int H, int T, int d, int recon, int ste,
                 int causal) {
  const bool ol = need_ol(recon, ste);
  char *b = static_cast<char *>(base);
  auto at = [&](int f) { return b + field_offset(B, H, T, d, recon, ste, causal, f); };
  Stats s;
  s.M = (float *)at(KIA_STAT_M);
  s.m = (float *)at(KIA_STAT_m);
  s.W = (float *)at(KIA_STAT_W);
  s.WL = (float *)at(KIA_STAT_WL);
  s.amax = (int *)at(KIA_STAT_AMAX);
  s.amin = (int *)at(KIA_STAT_AMIN);
  s.nmax = (int *)at(KIA_STAT_NMAX);
  s.nmin = (int *)at(KIA_STAT_NMIN);
  s.rowrec = (float *)at(KIA_STAT_ROWREC);
  s.sself = (float *)at(KIA_STAT_SSELF);
  s.cM = (float *)at(KIA_STAT_CM);
  s.OL = ol ? (float *)at(KIA_STAT_OL) : nullptr;
  s.dS = (float *)at(KIA_STAT_DS);
  s.U = (float *)at(KIA_STAT_U);
  s.part = (float *)at(KIA_STAT_PART);
  return s;
}

float softmax_scale(int d) { return (float)(1.0 / sqrt((double)d)); }

int g_grid = KIA_GRID_AUTO;  // kia_set_grid_policy
int g_det = 0;               // kia_set_deterministic

// Compute units of the current device (queried once per device).
int device_cus() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cached[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        n <= 0)
      n = 256;
    cached[dev] = n;
  }
  return cached[dev];
}

// ---- launch timing hook (kia_timing_enable / kia_timing_read) -----------
struct TimedLaunch {
  const char *name;
  hipEvent_t start, stop;
};
bool g_timing = false;
std::vector<TimedLaunch> g_launches;

void clear_launches() {
  for (auto &t : g_launches) {
    hipEventDestroy(t.start);
    hipEventDestroy(t.stop);
  }
  g_launches.clear();
}

// Runs `launch` (one kernel launch on stream s); when timing is on, brackets
// it with two events recorded on the same stream.
template <class F>
void timed(const char *name, hipStream_t s, F launch) {
  if (!g_timing || g_launches.size() >= 65536) {
    launch();
    return;
  }
  TimedLaunch t{name, nullptr, nullptr};
  if (hipEventCreate(&t.start) != hipSuccess || hipEventCreate(&t.stop) != hipSuccess) {
    launch();
    return;
  }
  hipEventRecord(t.start, s);
  launch();
  hipEventRecord(t.stop, s);
  g_launches.push_back(t);
}

int launched() {
  return hipGetLastError() == hipSuccess ? KIA_OK : KIA_ERR_HIP;
}

template <typename TI, int D, int CALIB, int RG, int KP>
void launch_fwd_k(const FwdArgsT<TI> &a, hipStream_t s) {
  const dim3 grid(a.BH * ((a.T + 32 * RG - 1) / (32 * RG))), block(64 * RG * KP);
  if constexpr (sizeof(TI) == 4) {
    if (is_exp_rec(a.recon)) {
      if (a.recon == KIA_RECON_SOFTMAX)
        hipLaunchKernelGGL((fwd_kernel<TI, D, CAL_FWM, REC_SOFTMAX, false, RG, KP>), grid, block, 0, s, a);
      else if (a.recon == KIA_RECON_BF16EXP)
        hipLaunchKernelGGL((fwd_kernel<TI, D, CAL_FWM, REC_BF16EXP, false, RG, KP>), grid, block, 0, s, a);
      else
        hipLaunchKernelGGL((fwd_kernel<TI, D, CAL_FWM, REC_FP8EXP, false, RG, KP>), grid, block, 0, s, a);
      return;
    }
  }
  if (a.recon == KIA_RECON_LERP)
    hipLaunchKernelGGL((fwd_kernel<TI, D, CALIB, REC_LERP, false, RG, KP>), grid, block, 0, s, a);
  else if (a.st.OL)
    hipLaunchKernelGGL((fwd_kernel<TI, D, CALIB, REC_NEAREST, true, RG, KP>), grid, block, 0, s, a);
  else
    hipLaunchKernelGGL((fwd_kernel<TI, D, CALIB, REC_NEAREST, false, RG, KP>), grid, block, 0, s, a);
}

// Launch shape by the number of 128-row blocks. On large grids 128 rows share each
// staged tile; below, row groups are given up for key parts, so that the longest
// causal row's keys are spread over two, four or eight waves and there are enough
// workgroups. Measured at T = 1024, FWM with Nearest and Prob-STE, a training
// forward (us; 1 x 8 / 1 x 4 / 2 x 2 / 4 x 1):
//   fp32 d = 16   96 blocks 29 / 31 / 54 / 98, 320 74 / 62 / 66 / 104,
//                 512 112 / 86 / 92 / 108, 768 - / 123 / 124 / 131
//   fp32 d = 32   96 blocks 33 / 37 / 59 / 113, 320 88 / 71 / 69 / 124,
//                 512 132 / 102 / 102 / 138, 768 - / 147 / 139 / 163
//   fp32 d = 64   96 blocks 48 / 52 / 80 / 135, 320 128 / 99 / 96 / 147,
//                 512 191 / 143 / 141 / 155, 768 - / 218 / 190 / 197
//   fp32 d = 128  96 blocks - / 79 / 120 / 209, 192 - / 148 / 128 / 213,
//                 512 - / 346 / 273 / 255
//   bf16 d = 64   96 blocks - / 26 / 40 / 66, 320 - / 48 / 44 / 69, 768 - / 92 / 78 / 78
//   bf16 d = 128  96 blocks - / 45 / 61 / 86, 192 - / 72 / 61 / 88, 768 - / 270 / 140 / 111
// Up to three blocks per CU 4 x 1 leaves its second round half empty. One 1 x 4
// workgroup fills a CU's LDS with fp32 V or with O and O_l sums at d = 128
// (`alone`); without O_l bf16 Nearest would gain from it up to one block per CU (192
// blocks 40 / 48), but the shape sets the order of the sums, and surrogate and
// gradient mode leave the forward's bits as they are: the rule looks at neither.
// Eight parts need more than four key tiles.
template <typename TI, int D, int CALIB>
void launch_fwd_c(const FwdArgsT<TI> &a, hipStream_t s) {
  constexpr bool F32 = sizeof(TI) == 4;
  const long blocks = (long)a.BH * ((a.T + 127) / 128), cus = device_cus();
  const bool split = g_grid == KIA_GRID_SPLIT, autog = g_grid == KIA_GRID_AUTO;
  if constexpr (F32 && D <= 64) {
    if (split || (autog && blocks <= cus / 2 && a.T > 128))
      return launch_fwd_k<TI, D, CALIB, 1, 8>(a, s);
  }
  const bool alone = a.recon == KIA_RECON_NEAREST
                         ? FwdShape<TI, D, REC_NEAREST, true, 1, 4>::OCC == 1
                         : FwdShape<TI, D, REC_LERP, false, 1, 4>::OCC == 1;
  const long most14 = alone ? cus / 2 : F32 && D == 16 ? 2 * cus : cus;
  const long most22 = D == 128 ? 2 * cus : 3 * cus;
  if (split || (autog && blocks <= most14)) return launch_fwd_k<TI, D, CALIB, 1, 4>(a, s);
  if (autog && blocks <= most22) return launch_fwd_k<TI, D, CALIB, 2, 2>(a, s);
  launch_fwd_k<TI, D, CALIB, 4, 1>(a, s);
}

template <typename TI, int D>
void launch_fwd(const FwdArgsT<TI> &a, hipStream_t s) {
  timed("kia_fwd", s, [&] {
    if (a.calib == KIA_CALIB_MINMAX) launch_fwd_c<TI, D, CAL_MINMAX>(a, s);
    else if (a.calib == KIA_CALIB_RESOLVED) launch_fwd_c<TI, D, CAL_RESOLVED>(a, s);
    else launch_fwd_c<TI, D, CAL_FWM>(a, s);
  });
}

template <int D, typename TI>
void launch_codes(const CodesArgsT<TI> &a, int recon, hipStream_t s) {
  const dim3 grid(a.BH * ((a.T + 127) / 128)), block(256);
  timed("kia_codes", s, [&] {
    if constexpr (sizeof(TI) == 4) {
      if (recon == KIA_RECON_SOFTMAX) {
        hipLaunchKernelGGL((codes_kernel<D, CAL_FWM, REC_SOFTMAX, TI>), grid, block, 0, s, a);
        return;
      }
      if (recon == KIA_RECON_BF16EXP) {
        hipLaunchKernelGGL((codes_kernel<D, CAL_FWM, REC_BF16EXP, TI>), grid, block, 0, s, a);
        return;
      }
      if (recon == KIA_RECON_FP8EXP) {
        hipLaunchKernelGGL((codes_kernel<D, CAL_FWM, REC_FP8EXP, TI>), grid, block, 0, s, a);
        return;
      }
    }
    if (a.calib == KIA_CALIB_MINMAX)
      hipLaunchKernelGGL((codes_kernel<D, CAL_MINMAX, REC_LERP, TI>), grid, block, 0, s, a);
    else if (a.calib == KIA_CALIB_RESOLVED)
      hipLaunchKernelGGL((codes_kernel<D, CAL_RESOLVED, REC_LERP, TI>), grid, block, 0, s, a);
    else
      hipLaunchKernelGGL((codes_kernel<D, CAL_FWM, REC_LERP, TI>), grid, block, 0, s, a);
  });
}

// ---- backward ------------------------------------------------------------
template <typename TI, int D, int CALIB, int RECON>
void launch_main(const BwdArgsT<TI> &a, int nkb, hipStream_t s) {
  hipLaunchKernelGGL((bwd_main_kernel<TI, D, CALIB, RECON>), dim3(a.BH * nkb), dim3(256), 0, s, a);
}
template <typename TI, int D, int CALIB>
void launch_main_c(const BwdArgsT<TI> &a, int nkb, hipStream_t s) {
  if (a.recon == KIA_RECON_LERP) launch_main<TI, D, CALIB, REC_LERP>(a, nkb, s);
  else launch_main<TI, D, CALIB, REC_NEAREST>(a, nkb, s);
}

// The backward's launches: pre-pass, main, dQ and, by gradient mode, ties or
// the P1 projection. Every kernel is one template over the input type TI.
template <int D, typename TI>
void launch_bwd(const BwdArgsT<TI> &a, hipStream_t s) {
  constexpr bool B16 = sizeof(TI) == 2;
  const size_t R = (size_t)a.BH * a.T;
  const size_t rpb = 256 / (D / 4);
  timed("kia_bwd_pre", s, [&] {
    hipLaunchKernelGGL((bwd_pre_kernel<D, TI>), dim3((unsigned)((R + rpb - 1) / rpb)),
                       dim3(256), 0, s, a);
  });
  const int nkb = (a.T + 127) / 128 * a.qsplit;
  timed("kia_bwd_main", s, [&] {
    if constexpr (!B16) {
      if (a.recon == KIA_RECON_SOFTMAX) return launch_main<TI, D, CAL_FWM, REC_SOFTMAX>(a, nkb, s);
      if (a.recon == KIA_RECON_BF16EXP) return launch_main<TI, D, CAL_FWM, REC_BF16EXP>(a, nkb, s);
      if (a.recon == KIA_RECON_FP8EXP) return launch_main<TI, D, CAL_FWM, REC_FP8EXP>(a, nkb, s);
    }
    if (a.calib == KIA_CALIB_MINMAX) launch_main_c<TI, D, CAL_MINMAX>(a, nkb, s);
    else if (a.calib == KIA_CALIB_RESOLVED) launch_main_c<TI, D, CAL_RESOLVED>(a, nkb, s);
    else launch_main_c<TI, D, CAL_FWM>(a, nkb, s);
  });
  // deterministic backward: the key blocks' row-sum partials added up in
  // order (timed with the main kernel)
  if (a.det && a.grad != GRAD_DETACH) {
    timed("kia_bwd_main", s, [&] {
      hipLaunchKernelGGL(row_sums_kernel<TI>, dim3((unsigned)((R + 255) / 256)), dim3(256), 0,
                         s, a);
    });
  }
  const int nq = (a.T + 31) / 32;
  timed("kia_bwd_dq", s, [&] {
    constexpr int QG = dq_tiles(D);
    int items = 0;
    for (int g = 0; g < (nq + QG - 1) / QG; ++g)
      items += dq_pieces(g, a.T, a.causal, a.dq_piece, QG);
    hipLaunchKernelGGL((bwd_dq_kernel<TI, D, QG>), dim3(a.BH * items), dim3(128 * QG), 0, s, a);
    // deterministic backward: the unique extrema's calibration terms
    // gathered onto dK per 32 keys (bwd_dq leaves them out)
    // (four waves per 32 keys when the scans are long or the grid is
    // small, one otherwise: the four waves' 4x LDS halves the residency)
    if (a.det && grad_channels(a.grad)) {
      if (a.T >= 4096 || a.BH * nq < 8 * device_cus())
        hipLaunchKernelGGL((calib_gather_kernel<D, TI, 4>), dim3(a.BH * nq), dim3(256), 0, s, a);
      else
        hipLaunchKernelGGL((calib_gather_kernel<D, TI, 1>), dim3(a.BH * nq), dim3(64), 0, s, a);
    }
  });
  if (grad_channels(a.grad)) {
    // one wave per 32-row block, or per slice in the deterministic backward
    const size_t nw = a.det ? (size_t)a.BH : (size_t)a.BH * ((a.T + 31) / 32);
    timed("kia_bwd_ties", s, [&] {
      hipLaunchKernelGGL((bwd_ties_kernel<D, TI>), dim3((unsigned)((nw + 3) / 4)),
                         dim3(256), 0, s, a);
    });
  }
  if (a.grad == GRAD_P1) {
    timed("kia_bwd_p1", s, [&] {
      hipLaunchKernelGGL((bwd_p1_kernel<D, TI>), dim3(a.BH * ((D + 63) / 64)), dim3(256), 0,
                         s, a);
    });
  }
}

}  // namespace

extern "C" int kia_stats_bytes(int B, int H, int T, int d, int recon, int ste,
                               int causal, size_t *bytes) {
  if (!bytes) return KIA_ERR_NULL;
  *bytes = 0;
  int rc = check_shape(B, H, T, d);
  if (rc) return rc;
  if (!recon_ok(recon) || (ste != 0 && ste != 1) || (causal != 0 && causal != 1))
    return KIA_ERR_ENUM;
  rc = check_size(B, H, T, d, causal);
  if (rc) return rc;
  *bytes = field_offset(B, H, T, d, recon, ste, causal, NFIELD);
  return KIA_OK;
}

extern "C" int kia_stats_offset(int B, int H, int T, int d, int recon, int ste,
                                int causal, int field, size_t *offset) {
  if (!offset) return KIA_ERR_NULL;
  *offset = 0;
  int rc = check_shape(B, H, T, d);
  if (rc) return rc;
  if (!recon_ok(recon) || (ste != 0 && ste != 1) || (causal != 0 && causal != 1) ||
      field < 0 || field >= NFIELD)
    return KIA_ERR_ENUM;
  rc = check_size(B, H, T, d, causal);
  if (rc) return rc;
  *offset = field_offset(B, H, T, d, recon, ste, causal, field);
  return KIA_OK;
}

namespace {

// Outputs of the bf16-output variant (bf16 bits), or none.
struct Bf16Out {
  uint16_t *o = nullptr, *dq = nullptr, *dk = nullptr, *dv = nullptr;
};

size_t acc_offset(int B, int H, int T, int d, int causal) {
  return field_offset(B, H, T, d, 0, 0, causal, KIA_STAT_ACC);
}

template <typename TI>
int attn_fwd(const TI *q, const TI *k, const TI *v, float *o, void *stats, int B, int H, int T,
             int d, int K, int calib, float tau, int recon, int ste, int detach, int causal,
             void *stream, const Bf16Out *bo = nullptr) {
  int rc = check_args(B, H, T, d, K, calib, tau, recon, ste, detach, causal);
  if (rc) return rc;
  if (sizeof(TI) == 2 && is_exp_rec(recon)) return KIA_ERR_ENUM;  // fp32 inputs only
  if (bo) o = reinterpret_cast<float *>(bo->o);  // never written as fp32
  if (!q || !k || !v || !o || !stats) return KIA_ERR_NULL;
  if (!al16(q) || !al16(k) || !al16(v) || !al16(o) || !al256(stats))
    return KIA_ERR_ALIGN;
  FwdArgsT<TI> a;
  a.q = q; a.k = k; a.v = v; a.o = o;
  if (bo) a.o16 = bo->o;
  a.st = make_stats(stats, B, H, T, d, recon, ste, causal);
  if (detach == KIA_GRAD_NONE) {  // only the backward reads O^L and the stored decisions
    a.st.OL = nullptr;
    a.keep = 0;
  }
  a.BH = B * H; a.T = T; a.K = K; a.calib = calib; a.recon = recon;
  a.causal = causal; a.tau = calib != KIA_CALIB_MINMAX ? tau : 0.f;
  if (is_exp_rec(recon)) { a.calib = CAL_FWM; a.tau = 0.f; a.K = 1; }  // maximum only
  a.scale = softmax_scale(d);
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (a.calib != CAL_MINMAX && !is_exp_rec(recon)) {
    const double h = (double)a.tau / K, LOG2E = 1.4426950408889634074;
    a.gc = K / (double)a.tau;
    a.ga = (float)(a.gc * (double)a.scale);
    a.ghl = (float)(h * LOG2E);
    a.gb1l = (float)((h - (double)a.tau) * LOG2E);
    a.gemh = (float)exp(-h);
  }
  switch (d) {
    case 16: launch_fwd<TI, 16>(a, s); break;
    case 32: launch_fwd<TI, 32>(a, s); break;
    case 64: launch_fwd<TI, 64>(a, s); break;
    default: launch_fwd<TI, 128>(a, s); break;
  }
  return launched();
}

// Parts into which the main kernel splits each key block's query range. A
// split shortens the longest workgroup (the causal key block 0, with L query
// tiles) until the tiles are spread over the chip's slots, and each part adds
// its dK and dV atomically: about 0.05 us a part over the whole chip at
// d = 64, 0.02 of a tile's time with fp32 inputs and 0.035 with bf16. The
// least of L / n + cost n blocks is n = sqrt(L / (cost blocks)). Measured (us;
// 1 / 2 / 3 / 4 / 6 parts) at T = 1024, d = 64: fp32 96 blocks 99 / 55 / 44 /
// 39 / 47, 192 blocks 100 / 63 / 55 / 67 / 86, 320 blocks 105 / 75 / 90; bf16
// 96 blocks 50 / 30 / 25 / 28, 192 blocks 51 / 34 / 41; T = 4096, 256 blocks
// 399 / 255 / 201 / 199 / 212; bf16 T = 8192 d = 128, 256 blocks 726 / 438 /
// 336 / 326 / 349.
int main_parts(int BH, int T, int d, bool f32, int causal) {
  if (g_grid == KIA_GRID_WIDE) return 1;
  const double blocks = (double)BH * ((T + 127) / 128), L = (T + 31) / 32;
  const double slots = device_cus() * (f32 && d == 128 ? 1.0 : 2.0);
  const double cost = (f32 ? 0.02 : 0.035) * std::min(d, 80) / 64.0;
  // no further than the point where every slot is busy throughout, nor than one
  // query tile a part
  const double most = std::min(L, std::ceil((causal ? 2.0 : 1.0) * slots / blocks));
  // (from one block per CU up four at most, see BwdArgsT::fold)
  const double cap = blocks < device_cus() ? 8.0 : 4.0;
  int n = (int)std::min(cap, std::min(most, std::floor(std::sqrt(L / (cost * blocks)) + 0.5)));
  return std::max(n, g_grid == KIA_GRID_SPLIT ? 2 : 1);
}

template <typename TI>
int attn_bwd(const TI *q, const TI *k, const TI *v, const float *o, const TI *dO,
             void *stats, float *dq, float *dk, float *dv, int B, int H, int T, int d, int K,
             int calib, float tau, int recon, int ste, int detach, int causal,
             void *stream, const Bf16Out *bo = nullptr) {
  int rc = check_args(B, H, T, d, K, calib, tau, recon, ste, detach, causal);
  if (rc) return rc;
  if (detach == KIA_GRAD_NONE) return KIA_ERR_ENUM;  // forward only
  if (sizeof(TI) == 2 && is_exp_rec(recon)) return KIA_ERR_ENUM;  // fp32 inputs only
  if (bo) {
    // bf16 outputs: dQ and dK accumulate in fp32 in the stats field ACC
    // (rounded once at the end), dV is written as bf16 by the main kernel
    o = reinterpret_cast<const float *>(bo->o);
    dv = reinterpret_cast<float *>(bo->dv);
    if (!bo->dq || !bo->dk || !stats) return KIA_ERR_NULL;
    if (!al16(bo->dq) || !al16(bo->dk) || !al256(stats)) return KIA_ERR_ALIGN;
    dq = reinterpret_cast<float *>(static_cast<char *>(stats) + acc_offset(B, H, T, d, causal));
    dk = dq + (size_t)B * H * T * d;
    // dV as bf16 straight from the main kernel, or (split main kernel, whose
    // parts add up atomically) through the third fp32 accumulator
    if (!bo->dv) return KIA_ERR_NULL;
    dv = dk + (size_t)B * H * T * d;
  }
  if (!q || !k || !v || !o || !dO || !stats || !dq || !dk || !dv)
    return KIA_ERR_NULL;
  if (!al16(q) || !al16(k) || !al16(v) || !al16(o) || !al16(dO) ||
      !al16(dq) || !al16(dk) || !al16(dv) || !al256(stats))
    return KIA_ERR_ALIGN;
  BwdArgsT<TI> a;
  a.q = q; a.k = k; a.v = v; a.o = o; a.dO = dO;
  a.dq = dq; a.dk = dk; a.dv = dv;
  if (bo) a.o16 = bo->o;
  a.st = make_stats(stats, B, H, T, d, recon, ste, causal);
  a.BH = B * H; a.T = T; a.K = K; a.calib = calib; a.recon = recon;
  a.ste = ste; a.grad = detach; a.causal = causal;
  a.qsplit = main_parts(B * H, T, d, sizeof(TI) == 4, causal);
  a.dq_piece = 0;
  if (g_grid != KIA_GRID_WIDE) {
    const bool force = g_grid == KIA_GRID_SPLIT;
    const int cus = device_cus();
    // dQ: groups of dq_tiles(d) query tiles; when they do not fill the chip,
    // their keys are cut into pieces so that there are about two per CU. A bf16
    // group at d = 128 takes its keys twice as fast as an fp32 one and a piece has
    // the same atomic epilogue: one piece per CU of at least eight chunks, and none
    // where the longest group has 16 chunks at most or three quarters of the CUs
    // have one. Measured there, FWM Nearest / MinMax LERP (us; none, eight chunks
    // at least, two per CU): B1 H24 T1024 27 / 37, 38 / 48, 47 / 59; B1 H14 T2048
    // 38 / 54, 53 / 71, -; B1 H4 T2048 37 / 44, 25 / 36, -; B1 H1 T8192 (17 chunks)
    // 102 / 114, 50 / 63, 59 / 70.
    const int qg = dq_tiles(d);
    const int npq = (T + 32 * qg - 1) / (32 * qg);
    const bool light = sizeof(TI) == 2 && d == 128;
    const int groups = B * H * npq, wanted = light ? cus : 2 * cus;
    const bool split = light ? 4 * groups < 3 * cus && dq_chunks(npq - 1, T, causal, qg) > 16
                             : groups < cus;
    if (split || force) {
      long chunks = 0;
      for (int g = 0; g < npq; ++g) chunks += dq_chunks(g, T, causal, qg);
      chunks *= (long)B * H;
      a.dq_piece = (int)std::max(light && !force ? 8L : 2L, (chunks + wanted - 1) / wanted);
    }
  }
  // from one 128-key block per CU up dV is bitwise repeatable: at most two parts
  // add into one buffer (the groups of the dQ kernel fill the chip there, so it
  // is free; not where the policy cuts them all the same)
  if (a.qsplit > 2 && (long)B * H * ((T + 127) / 128) >= device_cus()) {
    if (a.dq_piece > 0) a.qsplit = 2;
    else a.fold = 1;
  }
  // the deterministic backward takes the unsplit launch shapes
  if (g_det) { a.qsplit = 1; a.dq_piece = 0; a.fold = 0; a.det = 1; }
  if (bo && a.qsplit == 1) a.dv16 = bo->dv;
  a.tau = calib != KIA_CALIB_MINMAX ? tau : 0.f;
  if (is_exp_rec(recon)) { a.calib = CAL_FWM; a.tau = 0.f; a.K = 1; a.ste = STE_WEIGHT; }
  a.scale = softmax_scale(d);
  if (a.calib != CAL_MINMAX && !is_exp_rec(recon)) {
    const float h = a.tau / (float)K;
    a.ghl = h * 1.44269504f;
    a.gemh = expf(-h);
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  switch (d) {
    case 16: launch_bwd<16, TI>(a, s); break;
    case 32: launch_bwd<32, TI>(a, s); break;
    case 64: launch_bwd<64, TI>(a, s); break;
    default: launch_bwd<128, TI>(a, s); break;
  }
  if (bo) {
    const size_t n8 = (size_t)B * H * T * d / 8;
    timed("kia_cast_bf16", s, [&] {
      const dim3 grid((unsigned)((n8 + 255) / 256), a.dv16 ? 2 : 3), block(256);
      hipLaunchKernelGGL(cast_bf16_kernel, grid, block, 0, s, dq, bo->dq, bo->dk, bo->dv, n8);
    });
  }
  return launched();
}

template <typename TI>
int debug_codes(const TI *q, const TI *k, const void *stats, uint16_t *codes, int B, int H,
                int T, int d, int K, int calib, float tau, int recon, int causal,
                void *stream) {
  int rc = check_args(B, H, T, d, K, calib, tau, recon, 0, 0, causal);
  if (rc) return rc;
  if (sizeof(TI) == 2 && is_exp_rec(recon)) return KIA_ERR_ENUM;  // fp32 inputs only
  if (!q || !k || !stats || !codes) return KIA_ERR_NULL;
  if (!al16(q) || !al16(k) || !al256(stats)) return KIA_ERR_ALIGN;
  CodesArgsT<TI> a;
  a.q = q; a.k = k;
  a.st = make_stats(const_cast<void *>(stats), B, H, T, d, recon, 0, causal);
  a.codes = codes;
  a.BH = B * H; a.T = T; a.K = K; a.calib = calib; a.causal = causal;
  a.tau = calib != KIA_CALIB_MINMAX ? tau : 0.f;
  if (is_exp_rec(recon)) { a.calib = CAL_FWM; a.tau = 0.f; a.K = 1; }
  a.scale = softmax_scale(d);
  hipStream_t s = static_cast<hipStream_t>(stream);
  switch (d) {
    case 16: launch_codes<16, TI>(a, recon, s); break;
    case 32: launch_codes<32, TI>(a, recon, s); break;
    case 64: launch_codes<64, TI>(a, recon, s); break;
    default: launch_codes<128, TI>(a, recon, s); break;
  }
  return launched();
}

}  // namespace

extern "C" int kia_attn_fwd(const float *q, const float *k, const float *v,
                            float *o, void *stats, int B, int H, int T, int d,
                            int K, int calib, float tau, int recon, int ste,
                            int detach, int causal, void *stream) {
  return attn_fwd(q, k, v, o, stats, B, H, T, d, K, calib, tau, recon, ste, detach, causal,
                  stream);
}

extern "C" int kia_attn_bwd(const float *q, const float *k, const float *v,
                            const float *o, const float *dO, void *stats,
                            float *dq, float *dk, float *dv, int B, int H,
                            int T, int d, int K, int calib, float tau,
                            int recon, int ste, int detach, int causal,
                            void *stream) {
  return attn_bwd(q, k, v, o, dO, stats, dq, dk, dv, B, H, T, d, K, calib, tau, recon, ste,
                  detach, causal, stream);
}

// ---- static scratch of kia_attn_fwd_bwd_static ---------------------------
// The statistics of the no-allocation entry point live in this array; every
// GPU the library runs on holds its own copy until the process ends. In host
// code `scratch` only names the symbol: its device address on the current
// GPU comes from hipGetSymbolAddress, taken once per device (scratch_base).
static __device__ __align__(256) unsigned char scratch[KIA_STATIC_BYTES];

namespace {
std::mutex g_scratch_mu;
void *g_scratch_ptr[64] = {};

int scratch_base(void **out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return KIA_ERR_HIP;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return KIA_ERR_HIP;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return KIA_OK;
}
}  // namespace

extern "C" int kia_attn_fwd_bwd_static(const float *q, const float *k, const float *v,
                                       const float *dO, float *o, float *dq, float *dk,
                                       float *dv, int B, int H, int T, int d, int K,
                                       int calib, float tau, int recon, int ste, int detach,
                                       int causal, void *stream) {
  int rc = check_args(B, H, T, d, K, calib, tau, recon, ste, detach, causal);
  if (rc) return rc;
  if (detach == KIA_GRAD_NONE) return KIA_ERR_ENUM;  // its backward needs the forward's state
  if (!q || !k || !v || !dO || !o || !dq || !dk || !dv) return KIA_ERR_NULL;
  if (!al16(q) || !al16(k) || !al16(v) || !al16(dO) || !al16(o) || !al16(dq) || !al16(dk) ||
      !al16(dv))
    return KIA_ERR_ALIGN;
  if (field_offset(B, H, T, d, recon, ste, causal, NFIELD) > (size_t)KIA_STATIC_BYTES)
    return KIA_ERR_SCRATCH;
  void *base = nullptr;
  rc = scratch_base(&base);
  if (rc) return rc;
  rc = attn_fwd(q, k, v, o, base, B, H, T, d, K, calib, tau, recon, ste, detach, causal,
                stream);
  if (rc) return rc;
  return attn_bwd(q, k, v, o, dO, base, dq, dk, dv, B, H, T, d, K, calib, tau, recon, ste,
                  detach, causal, stream);
}

extern "C" int kia_debug_codes(const float *q, const float *k,
                               const void *stats, uint16_t *codes, int B,
                               int H, int T, int d, int K, int calib,
                               float tau, int recon, int causal,
                               void *stream) {
  return debug_codes(q, k, stats, codes, B, H, T, d, K, calib, tau, recon, causal, stream);
}

extern "C" int kia_attn_fwd_bf16(const uint16_t *q, const uint16_t *k, const uint16_t *v,
                                 float *o, void *stats, int B, int H, int T, int d,
                                 int K, int calib, float tau, int recon, int ste,
                                 int detach, int causal, void *stream) {
  return attn_fwd(q, k, v, o, stats, B, H, T, d, K, calib, tau, recon, ste, detach, causal,
                  stream);
}

extern "C" int kia_attn_bwd_bf16(const uint16_t *q, const uint16_t *k, const uint16_t *v,
                                 const float *o, const uint16_t *dO, void *stats,
                                 float *dq, float *dk, float *dv, int B, int H,
                                 int T, int d, int K, int calib, float tau,
                                 int recon, int ste, int detach, int causal,
                                 void *stream) {
  return attn_bwd(q, k, v, o, dO, stats, dq, dk, dv, B, H, T, d, K, calib, tau, recon, ste,
                  detach, causal, stream);
}

extern "C" int kia_stats_bytes_bf16o(int B, int H, int T, int d, int recon, int ste,
                                     int causal, size_t *bytes) {
  int rc = kia_stats_bytes(B, H, T, d, recon, ste, causal, bytes);
  if (rc) return rc;
  *bytes = acc_offset(B, H, T, d, causal) + align256((size_t)3 * B * H * T * d * sizeof(float));
  return KIA_OK;
}

extern "C" int kia_attn_fwd_bf16o(const uint16_t *q, const uint16_t *k, const uint16_t *v,
                                  uint16_t *o, void *stats, int B, int H, int T, int d, int K,
                                  int calib, float tau, int recon, int ste, int detach,
                                  int causal, void *stream) {
  Bf16Out bo;
  bo.o = o;
  return attn_fwd(q, k, v, nullptr, stats, B, H, T, d, K, calib, tau, recon, ste, detach,
                  causal, stream, &bo);
}

extern "C" int kia_attn_bwd_bf16o(const uint16_t *q, const uint16_t *k, const uint16_t *v,
                                  const uint16_t *o, const uint16_t *dO, void *stats,
                                  uint16_t *dq, uint16_t *dk, uint16_t *dv, int B, int H, int T,
                                  int d, int K, int calib, float tau, int recon, int ste,
                                  int detach, int causal, void *stream) {
  Bf16Out bo;
  bo.o = const_cast<uint16_t *>(o);
  bo.dq = dq; bo.dk = dk; bo.dv = dv;
  return attn_bwd(q, k, v, nullptr, dO, stats, nullptr, nullptr, nullptr, B, H, T, d, K, calib,
                  tau, recon, ste, detach, causal, stream, &bo);
}

extern "C" int kia_debug_codes_bf16(const uint16_t *q, const uint16_t *k,
                                    const void *stats, uint16_t *codes, int B,
                                    int H, int T, int d, int K, int calib,
                                    float tau, int recon, int causal,
                                    void *stream) {
  return debug_codes(q, k, stats, codes, B, H, T, d, K, calib, tau, recon, causal, stream);
}

extern "C" int kia_debug_codes_stored(const void *stats, uint16_t *codes, int B, int H,
                                      int T, int d, int K, int calib, float tau, int recon,
                                      int ste, int causal, void *stream) {
  int rc = check_args(B, H, T, d, K, calib, tau, recon, ste, 0, causal);
  if (rc) return rc;
  if (!stats || !codes) return KIA_ERR_NULL;
  if (!al256(stats) || !al16(codes)) return KIA_ERR_ALIGN;
  if ((long double)B * H * T * T >= 9.2e18L) return KIA_ERR_SHAPE;
  StoredCodesArgs a;
  a.st = make_stats(const_cast<void *>(stats), B, H, T, d, recon, ste, causal);
  a.codes = codes;
  a.BH = B * H; a.T = T; a.K = K; a.causal = causal;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const size_t nw = (size_t)a.BH * ((T + 31) / 32);
  const dim3 grid((unsigned)((nw + 3) / 4)), block(256);
  timed("kia_codes_stored", s, [&] {
    if (recon == KIA_RECON_SOFTMAX)
      hipLaunchKernelGGL((stored_codes_kernel<CAL_FWM, REC_SOFTMAX>), grid, block, 0, s, a);
    else if (recon == KIA_RECON_BF16EXP)
      hipLaunchKernelGGL((stored_codes_kernel<CAL_FWM, REC_BF16EXP>), grid, block, 0, s, a);
    else if (recon == KIA_RECON_FP8EXP)
      hipLaunchKernelGGL((stored_codes_kernel<CAL_FWM, REC_FP8EXP>), grid, block, 0, s, a);
    else if (calib == KIA_CALIB_MINMAX)
      hipLaunchKernelGGL((stored_codes_kernel<CAL_MINMAX, REC_LERP>), grid, block, 0, s, a);
    else if (calib == KIA_CALIB_RESOLVED)
      hipLaunchKernelGGL((stored_codes_kernel<CAL_RESOLVED, REC_LERP>), grid, block, 0, s, a);
    else if (recon == KIA_RECON_NEAREST)  // compact one-byte codes
      hipLaunchKernelGGL((stored_codes_kernel<CAL_FWM, REC_NEAREST>), grid, block, 0, s, a);
    else
      hipLaunchKernelGGL((stored_codes_kernel<CAL_FWM, REC_LERP>), grid, block, 0, s, a);
  });
  return launched();
}

namespace {
template <typename TI>
int debug_scores(const TI *q, const TI *k, float *scores, int B, int H, int T, int d,
                 int causal, void *stream) {
  int rc = check_shape(B, H, T, d);
  if (rc) return rc;
  if (causal != 0 && causal != 1) return KIA_ERR_ENUM;
  if (!q || !k || !scores) return KIA_ERR_NULL;
  if (!al16(q) || !al16(k) || !al16(scores)) return KIA_ERR_ALIGN;
  if ((long double)B * H * T * T >= 9.2e18L) return KIA_ERR_SHAPE;
  ScoresArgsT<TI> a;
  a.q = q; a.k = k; a.scores = scores;
  a.BH = B * H; a.T = T; a.causal = causal;
  a.scale = softmax_scale(d);
  hipStream_t s = static_cast<hipStream_t>(stream);
  const dim3 grid(a.BH * ((T + 127) / 128)), block(256);
  timed("kia_scores", s, [&] {
    switch (d) {
      case 16: hipLaunchKernelGGL((scores_kernel<16, TI>), grid, block, 0, s, a); break;
      case 32: hipLaunchKernelGGL((scores_kernel<32, TI>), grid, block, 0, s, a); break;
      case 64: hipLaunchKernelGGL((scores_kernel<64, TI>), grid, block, 0, s, a); break;
      default: hipLaunchKernelGGL((scores_kernel<128, TI>), grid, block, 0, s, a); break;
    }
  });
  return launched();
}
}  // namespace

extern "C" int kia_debug_scores(const float *q, const float *k, float *scores, int B, int H,
                                int T, int d, int causal, void *stream) {
  return debug_scores(q, k, scores, B, H, T, d, causal, stream);
}

extern "C" int kia_debug_scores_bf16(const uint16_t *q, const uint16_t *k, float *scores,
                                     int B, int H, int T, int d, int causal, void *stream) {
  return debug_scores(q, k, scores, B, H, T, d, causal, stream);
}

extern "C" int kia_debug_score_grad(const void *stats, int input_bf16, float *g_self,
                                    float *cM, float *cm, int B, int H, int T, int d,
                                    int calib, int recon, int ste, int causal,
                                    void *stream) {
  int rc = check_shape(B, H, T, d);
  if (rc) return rc;
  if (calib < KIA_CALIB_MINMAX || calib > KIA_CALIB_RESOLVED || !recon_ok(recon) ||
      (ste != 0 && ste != 1) ||
      (causal != 0 && causal != 1) || (input_bf16 != 0 && input_bf16 != 1) ||
      (input_bf16 && is_exp_rec(recon)))
    return KIA_ERR_ENUM;
  if (is_exp_rec(recon)) calib = KIA_CALIB_FWM;  // maximum only
  if (!stats || !g_self || !cM || !cm) return KIA_ERR_NULL;
  if (!al256(stats) || !al16(g_self) || !al16(cM) || !al16(cm)) return KIA_ERR_ALIGN;
  if ((long double)B * H * T * T >= 9.2e18L) return KIA_ERR_SHAPE;
  GradArgs a;
  a.st = make_stats(const_cast<void *>(stats), B, H, T, d, recon, ste, causal);
  a.g_self = g_self; a.cM = cM; a.cm = cm;
  a.BH = B * H; a.T = T; a.calib = calib; a.causal = causal; a.bf16 = input_bf16;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const size_t nw = (size_t)a.BH * ((T + 31) / 32);
  timed("kia_score_grad", s, [&] {
    hipLaunchKernelGGL(score_grad_kernel, dim3((unsigned)((nw + 3) / 4)), dim3(256), 0, s, a);
  });
  return launched();
}

namespace {
template <int D, int CALIB, int RECON>
void launch_geo_c(const GeoArgs &a, hipStream_t s) {
  const dim3 grid(a.BH * ((a.T + 127) / 128)), block(256);
  // the quantile needs the order statistics floor((T-1)/1000) and the next
  const int need = (a.T - 1) / 1000 + 2;
  if (need <= 3)
    hipLaunchKernelGGL((geometry_kernel<D, CALIB, RECON, 3>), grid, block, 0, s, a);
  else if (need <= 12)
    hipLaunchKernelGGL((geometry_kernel<D, CALIB, RECON, 12>), grid, block, 0, s, a);
  else
    hipLaunchKernelGGL((geometry_kernel<D, CALIB, RECON, 67>), grid, block, 0, s, a);
}

template <int D>
void launch_geo(const GeoArgs &a, int calib, int recon, hipStream_t s) {
  timed("kia_geometry", s, [&] {
    if (calib == KIA_CALIB_MINMAX) {
      if (recon == KIA_RECON_LERP) launch_geo_c<D, CAL_MINMAX, REC_LERP>(a, s);
      else launch_geo_c<D, CAL_MINMAX, REC_NEAREST>(a, s);
    } else {
      if (recon == KIA_RECON_LERP) launch_geo_c<D, CAL_FWM, REC_LERP>(a, s);
      else launch_geo_c<D, CAL_FWM, REC_NEAREST>(a, s);
    }
  });
}
}  // namespace

extern "C" int kia_geometry_probe(const float *q, const float *k, const void *stats,
                                  float *out, int B, int H, int T, int d, int K,
                                  int calib, float tau, int recon, int causal,
                                  void *stream) {
  int rc = check_args(B, H, T, d, K, calib, tau, recon, 0, 0, causal);
  if (rc) return rc;
  if (calib == KIA_CALIB_RESOLVED || is_exp_rec(recon)) return KIA_ERR_ENUM;
  if (!q || !k || !stats || !out) return KIA_ERR_NULL;
  if (!al16(q) || !al16(k) || !al16(out) || !al256(stats)) return KIA_ERR_ALIGN;
  GeoArgs a;
  a.q = q; a.k = k;
  a.st = make_stats(const_cast<void *>(stats), B, H, T, d, recon, 0, causal);
  a.out = out;
  a.BH = B * H; a.T = T; a.K = K; a.causal = causal;
  a.tau = calib == KIA_CALIB_FWM ? tau : 0.f;
  a.scale = softmax_scale(d);
  hipStream_t s = static_cast<hipStream_t>(stream);
  switch (d) {
    case 16: launch_geo<16>(a, calib, recon, s); break;
    case 32: launch_geo<32>(a, calib, recon, s); break;
    case 64: launch_geo<64>(a, calib, recon, s); break;
    default: launch_geo<128>(a, calib, recon, s); break;
  }
  return launched();
}

extern "C" int kia_mfma_peak_probe(unsigned long long *out, int workgroups, int iters,
                                   void *stream) {
  if (!out) return KIA_ERR_NULL;
  if ((reinterpret_cast<uintptr_t>(out) & 7) != 0) return KIA_ERR_ALIGN;
  if (workgroups < 1 || workgroups > (1 << 20) || iters < 1 || iters > (1 << 20))
    return KIA_ERR_SHAPE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  timed("kia_mfma_probe", s, [&] {
    hipLaunchKernelGGL(mfma_probe_kernel, dim3(workgroups), dim3(256), 0, s, out, iters);
  });
  return launched();
}

extern "C" int kia_set_deterministic(int on) {
  if (on != 0 && on != 1) return KIA_ERR_ENUM;
  g_det = on;
  return KIA_OK;
}

extern "C" int kia_set_grid_policy(int policy) {
  if (policy != KIA_GRID_AUTO && policy != KIA_GRID_WIDE && policy != KIA_GRID_SPLIT)
    return KIA_ERR_ENUM;
  g_grid = policy;
  return KIA_OK;
}

extern "C" int kia_timing_enable(int on) {
  clear_launches();
  g_timing = on != 0;
  return KIA_OK;
}

extern "C" int kia_timing_read(const char *name, double *total_ms,
                               int *launches) {
  if (!name || !total_ms || !launches) return KIA_ERR_NULL;
  *total_ms = 0.0;
  *launches = 0;
  for (auto &t : g_launches) {
    if (strcmp(t.name, name) != 0) continue;
    if (hipEventSynchronize(t.stop) != hipSuccess) return KIA_ERR_HIP;
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, t.start, t.stop) != hipSuccess) return KIA_ERR_HIP;
    *total_ms += ms;
    *launches += 1;
  }
  return KIA_OK;
}

extern "C" const char *kia_strerror(int code) {
  switch (code) {
    case KIA_OK: return "success";
    case KIA_ERR_NULL: return "a required pointer is NULL";
    case KIA_ERR_SHAPE: return "B, H or T out of range, or tensor size overflow";
    case KIA_ERR_HEADDIM: return "head dimension d must be 16, 32, 64 or 128";
    case KIA_ERR_K: return "K must lie in [1, 64]";
    case KIA_ERR_ENUM: return "calib/recon/ste/detach (gradient mode)/causal/field out of range";
    case KIA_ERR_TAU: return "FWM needs a finite tau > 0";
    case KIA_ERR_ALIGN: return "tensors must be 16-byte and stats 256-byte aligned";
    case KIA_ERR_HIP: return "HIP kernel launch failed";
    case KIA_ERR_SCRATCH:
      return "the problem's statistics exceed the static scratch of kia_attn_fwd_bwd_static "
             "(KIA_STATIC_BYTES)";
    default: return "unknown error code";
  }
}
