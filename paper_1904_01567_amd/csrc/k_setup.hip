// Case and batch set-up kernels: dose-rate matrix (Sec. 2.2.1 step (i)),
// its run-dtype copy, the default start time and the per-plan state.
#include "gmco_internal.h"

namespace gmco {
namespace {

// Round an FP32 value to BF16, nearest with ties to even (finite inputs).
__device__ inline uint16_t bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// Position of point r of a 32-point block in the BF16 / FP8 evaluation's transposed
// tile (its back-projection operand order): rows 4q .. 4q+3 and
// 16+4q .. 16+4q+3 of the block at positions 8q .. 8q+7.
__device__ inline int tpos32(int r) {
  return r < 16 ? 8 * (r >> 2) + (r & 3) : 8 * ((r - 16) >> 2) + 4 + ((r - 16) & 3);
}

// The dose-rate matrix and everything that is read off it, in one pass: per
// 32-point block a workgroup computes 64 columns at a time and writes
//   D64                the matrix in FP64 (every mode)
//   D32                its FP32 copy (all but DVH points)
//   D16, DT16          BF16 row-major, for the dose product (BF16 only), and
//                      dwell-major with the points of the block in the tile
//                      order above (BF16 and FP8)
//   colmax             the block's largest |D| per column (FP8: one row of
//                      the partial maxima of the column scales)
//   rowsum             sum over the columns of rows r0 .. r1 - 1, in column
//                      order (the start time's mean)
// so that the FP64 matrix is not read back.  Bound by the bytes written (16
// per element in BF16) and, close behind, by the FP64 square root and
// division: 42 us at 20,000 x 360 in BF16 (2.9 TB/s), where separate passes
// took 33 + 15 + 64 us, and 1,832 us for the start time by one workgroup with
// a row per thread; that case's load, weights and first evaluation of 1,000
// plans went from 2,609 to 708 us.
// Point-source law of the synthetic cases: (1 - 0.01 r) / max(r, 0.1 cm)^2.
// Rows follow the library's point order (grouped by structure): row i is the
// caller's point perm[i].  Padding rows and columns are zero.
enum { DOSE_D64 = 0, DOSE_F32 = 1, DOSE_BF16 = 2, DOSE_FP8 = 3 };
struct DoseArgs {
  const double* dwell;
  const double* pts;
  const double* user_D;
  const int* perm;
  int M, K, Mp, Kp, r0, r1;
  double* D64;
  float* D32;
  uint16_t* D16;
  uint16_t* DT16;
  double* colmax;  // [Mp / 32][Kp]
  double* rowsum;  // [Mp]
};

template <int MODE>
__global__ __launch_bounds__(256) void k_dose_matrix(DoseArgs a) {
  constexpr int NR = 32, NC = 64, RS = NC + 1;
  constexpr int TS = NR + 8;  // 80-byte rows: 16-byte aligned, the columns' writes spread over the banks
  __shared__ double sD[NR * RS];
  __shared__ __attribute__((aligned(16))) uint16_t sT[MODE >= DOSE_BF16 ? NC * TS : 8];
  __shared__ double sM[MODE == DOSE_FP8 ? 4 * NC : 1];
  const int i0 = blockIdx.x * NR;
  const int c = threadIdx.x & 63, w = threadIdx.x >> 6;  // column; rows 8 w .. 8 w + 7
  const bool sums = MODE != DOSE_D64 && i0 < a.r1 && i0 + NR > a.r0;
  double rs = 0.0;  // row i0 + threadIdx.x (first 32 threads)
  // the rows' points, the same for every chunk of columns (a wavefront's rows are uniform)
  int src[NR / 4];
#pragma unroll
  for (int k = 0; k < NR / 4; ++k) src[k] = i0 + 8 * w + k < a.M ? a.perm[i0 + 8 * w + k] : -1;
  for (int l0 = 0; l0 < a.Kp; l0 += NC) {
    const int l = l0 + c;
    const bool col = l < a.K;
    double dwx = 0.0, dwy = 0.0, dwz = 0.0, cm = 0.0;
    uint16_t t16[NR / 4] = {};
    if (col && a.user_D == nullptr) {
      dwx = a.dwell[3 * l + 0];
      dwy = a.dwell[3 * l + 1];
      dwz = a.dwell[3 * l + 2];
    }
#pragma unroll
    for (int k = 0; k < NR / 4; ++k) {
      const int r = 8 * w + k;
      double v = 0.0;
      if (src[k] >= 0 && col) {
        if (a.user_D != nullptr) {
          v = a.user_D[(size_t)src[k] * a.K + l];
        } else {
          const double dx = a.pts[3 * src[k] + 0] - dwx;
          const double dy = a.pts[3 * src[k] + 1] - dwy;
          const double dz = a.pts[3 * src[k] + 2] - dwz;
          const double r2 = sqrt(dx * dx + dy * dy + dz * dz);
          const double rc = r2 > 0.1 ? r2 : 0.1;
          v = (1.0 - 0.01 * r2) / (rc * rc);
        }
      }
      if (l < a.Kp) {
        const size_t at = (size_t)(i0 + r) * a.Kp + l;
        a.D64[at] = v;
        if constexpr (MODE >= DOSE_F32) a.D32[at] = (float)v;
        if constexpr (MODE >= DOSE_BF16) {
          const uint16_t h = bf16_rne((float)v);
          if constexpr (MODE == DOSE_BF16) a.D16[at] = h;
          t16[k] = h;
        }
      }
      if constexpr (MODE == DOSE_FP8) cm = fmax(cm, fabs(v));
      if (sums) sD[r * RS + c] = v;
    }
    if constexpr (MODE >= DOSE_BF16) {
      // rows 8 w .. 8 w + 3 and 8 w + 4 .. 8 w + 7 are runs of four positions
#pragma unroll
      for (int h = 0; h < 2; ++h)
        *reinterpret_cast<uint2*>(&sT[c * TS + tpos32(8 * w + 4 * h)]) =
            make_uint2(t16[4 * h] | (unsigned)t16[4 * h + 1] << 16, t16[4 * h + 2] | (unsigned)t16[4 * h + 3] << 16);
    }
    if constexpr (MODE == DOSE_FP8) sM[w * NC + c] = cm;
    if (MODE >= DOSE_BF16 || sums) __syncthreads();
    if constexpr (MODE >= DOSE_BF16) {
      // 64 bytes of a dwell's points by four threads
      const int lc = threadIdx.x >> 2, part = threadIdx.x & 3;
      if (l0 + lc < a.Kp)
        *reinterpret_cast<uint4*>(a.DT16 + (size_t)(l0 + lc) * a.Mp + i0 + 8 * part) =
            *reinterpret_cast<const uint4*>(&sT[lc * TS + 8 * part]);
    }
    if constexpr (MODE == DOSE_FP8) {
      if (threadIdx.x < NC && l < a.Kp)
        a.colmax[(size_t)blockIdx.x * a.Kp + l] =
            fmax(fmax(sM[c], sM[NC + c]), fmax(sM[2 * NC + c], sM[3 * NC + c]));
    }
    if (sums && threadIdx.x < NR) {
      const int n = min(NC, a.Kp - l0);  // 32 or 64
#pragma unroll 32
      for (int j = 0; j < n; ++j) rs += sD[threadIdx.x * RS + j];
    }
    if (MODE >= DOSE_BF16 || sums) __syncthreads();
  }
  if (sums && threadIdx.x < NR) a.rowsum[i0 + threadIdx.x] = rs;
}

// Per-dwell-column scale for the FP8 copy: s_l = max_i D_il / 224 (1 for an
// all-zero column), from the blocks' partial maxima.  A workgroup takes 64
// columns, its 16 wavefronts every 16th block.
__global__ __launch_bounds__(1024) void k_colscale(const double* __restrict__ colmax, int nb, int Kp,
                                                   float* __restrict__ cs) {
  __shared__ double red[16][64];
  const int c = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int l = blockIdx.x * 64 + c;
  double m = 0.0;
  if (l < Kp) {
#pragma unroll 8
    for (int b = w; b < nb; b += 16) m = fmax(m, colmax[(size_t)b * Kp + l]);
  }
  red[w][c] = m;
  __syncthreads();
  if (w > 0 || l >= Kp) return;
#pragma unroll
  for (int k = 1; k < 16; ++k) m = fmax(m, red[k][c]);
  cs[l] = m > 0.0 ? (float)(m / 224.0) : 1.f;
}

// FP8 (hardware e4m3 encoding) copy of D_il / s_l, row-major, four columns
// per thread.
__global__ void k_cast_fp8(const float* __restrict__ D32, size_t n4, int Kp4, const float* __restrict__ cs,
                           unsigned* __restrict__ D8) {
  for (size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x; idx < n4;
       idx += (size_t)gridDim.x * blockDim.x) {
    const float4 v = reinterpret_cast<const float4*>(D32)[idx];
    const float4 s = reinterpret_cast<const float4*>(cs)[idx % Kp4];
    const int lo = __builtin_amdgcn_cvt_pk_fp8_f32(v.x / s.x, v.y / s.y, 0, false);
    D8[idx] = (unsigned)__builtin_amdgcn_cvt_pk_fp8_f32(v.z / s.z, v.w / s.w, lo, true);
  }
}

// FP8 bytes widened to double with the column scale applied (for export).
__global__ void k_widen_fp8(const unsigned char* __restrict__ D8, const float* __restrict__ cs,
                            int Mp, int Kp, double* __restrict__ out) {
  const size_t n = (size_t)Mp * Kp;
  for (size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x; idx < n;
       idx += (size_t)gridDim.x * blockDim.x) {
    const size_t l = idx % Kp;
    out[idx] = (double)__builtin_amdgcn_cvt_f32_fp8((int)D8[idx], 0) * (double)cs[l];
  }
}

// t_bar = Rx / mean over the target rows of sum_l D_il, from the row sums:
// one workgroup, fixed summation order.
__global__ __launch_bounds__(1024) void k_start_time(const double* __restrict__ rowsum, int r0, int r1, double rx,
                                                     double* __restrict__ t_bar) {
  __shared__ double red[1024];
  double acc = 0.0;
#pragma unroll 8
  for (int i = r0 + threadIdx.x; i < r1; i += 1024) acc += rowsum[i];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int o = blockDim.x / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double mean = red[0] / (double)(r1 - r0);
    *t_bar = (r1 > r0 && mean > 0.0) ? rx / mean : 0.0;
  }
}

// Start point and weights of every plan slot.  Inactive slots (p >= P) get
// zero weights and the INACTIVE state.
// W is P x O hidden weights (one per organ); group j of organ gorg[j] gets
// w / N_pnt of its organ (eq. (obj)).
__global__ void k_init_plans(int P, int Pp, int K, int Kp, const double* __restrict__ t0,
                             const double* __restrict__ t_bar, const double* __restrict__ W,
                             int G, int O, const int* __restrict__ gorg,
                             const int* __restrict__ norm, float* __restrict__ xt,
                             float* __restrict__ x, float* __restrict__ wn,
                             double* __restrict__ W64, PlanState* __restrict__ ps) {
  const int p = blockIdx.x;
  if (p >= Pp) return;
  const bool live = p < P;
  const double tb = *t_bar;
  for (int l = threadIdx.x; l < Kp; l += blockDim.x) {
    float v = 0.f;
    if (live && l < K) {
      const double t = t0 ? t0[(size_t)p * K + l] : tb;
      v = (float)sqrt(t > 0.0 ? t : 0.0);
    }
    xt[(size_t)p * Kp + l] = v;
    x[(size_t)p * Kp + l] = v;
  }
  if (threadIdx.x < kGmax) {
    const int j = threadIdx.x;
    W64[(size_t)p * kGmax + j] = (live && j < O) ? W[(size_t)p * O + j] : 0.0;
    double w = 0.0;
    if (live && j < G) w = W[(size_t)p * O + gorg[j]];
    wn[(size_t)p * kGmax + j] = (j < G && norm[j] > 0) ? (float)(w / (double)norm[j]) : 0.f;
  }
  if (threadIdx.x == 0) {
    PlanState s;
    s.F = 0.0;
    s.Fprev = 0.0;
    s.alpha = 0.0;
    s.gtp = 0.0;
    s.status = live ? ST_INIT : ST_INACTIVE;
    s.iter = 0;
    s.ntrial = 0;
    s.hcount = 0;
    s.hhead = 0;
    s.nevals = 0;
    s.nevals0 = 0;
    s.pad = 0;
    ps[p] = s;
  }
}

// Dwell weights given by the caller (P x K) into the padded FP32 layout.  Bound
// by its trips to memory, so a row is one: four dwells a thread (Kp is at most
// 512), all its loads in flight, one 16-byte store.  Against a dwell per thread
// and trip, whole evaluate calls: 8 plans x 160 dwells 11.94 -> 11.68 us, 1 x 360
// 20.0 -> 19.7, 333 x 277 47.9 -> 47.4; 1,000 x 360 unchanged at 77.1.
template <class T>
__global__ __launch_bounds__(128) void k_x_to_device(const T* __restrict__ xin, int P, int K, int Kp,
                                                     float* __restrict__ xe) {
  const int p = blockIdx.x, l = 4 * (int)threadIdx.x;
  if (l >= Kp) return;
  T v[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) v[u] = xin[(size_t)min(p, P - 1) * K + min(l + u, K - 1)];
  float w[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) w[u] = (p < P && l + u < K) ? (float)v[u] : 0.f;
  *reinterpret_cast<float4*>(xe + (size_t)p * Kp + l) = make_float4(w[0], w[1], w[2], w[3]);
}

// Network inputs of the learned start: row p is the plan's hidden weights
// (one per organ, as given) followed by the case features.
__global__ void k_learned_inputs(const double* __restrict__ W64, const float* __restrict__ feat, int O,
                                 float* __restrict__ X) {
  const int p = blockIdx.x;
  const int n_in = O + 16 * O;
  for (int i = threadIdx.x; i < n_in; i += blockDim.x)
    X[(size_t)p * n_in + i] = i < O ? (float)W64[(size_t)p * kGmax + i] : feat[i - O];
}

// Start dwell weights from the network's output y (normalised by the uniform
// start): x0 = max(y, floor) sqrt(t_bar); a non-finite y stays non-finite, so
// that the plan's start objective is too and the plan falls back.
__global__ void k_learned_start(const float* __restrict__ Y, int K, int Kp, const double* __restrict__ t_bar,
                                float floor, float* __restrict__ xe) {
  const int p = blockIdx.x;
  const float sc = (float)sqrt(*t_bar);
  for (int l = threadIdx.x; l < Kp; l += blockDim.x) {
    float v = 0.f;
    if (l < K) {
      const float y = Y[(size_t)p * K + l];
      v = (isfinite(y) ? fmaxf(y, floor) : y) * sc;
    }
    xe[(size_t)p * Kp + l] = v;
  }
}

// Per plan: keep the learned start only where it is finite and its
// objective is below the uniform start's (plain L-BFGS from the uniform
// start is the fallback).  The start itself is checked, not only F: the
// penalty of eq. 1 as evaluated (min / max with the band edges) is 0 at a
// NaN dose.  The chosen point becomes the plan's start (status INIT).
__global__ void k_pick_start(const double* __restrict__ Fw, const double* __restrict__ Fu,
                             const float* __restrict__ xe, int Kp, float* __restrict__ x,
                             float* __restrict__ xt, int* __restrict__ n_warm, int* __restrict__ use_warm) {
  const int p = blockIdx.x;
  int bad = 0;
  for (int l = threadIdx.x; l < Kp; l += blockDim.x) bad |= !isfinite(xe[(size_t)p * Kp + l]);
  bad = __syncthreads_or(bad);
  const double fw = Fw[p];
  const bool warm = !bad && isfinite(fw) && fw < Fu[p];
  if (threadIdx.x == 0) {
    use_warm[p] = warm ? 1 : 0;
    if (warm) atomicAdd(n_warm, 1);
  }
  if (!warm) return;
  for (int l = threadIdx.x; l < Kp; l += blockDim.x) {
    const float v = xe[(size_t)p * Kp + l];
    x[(size_t)p * Kp + l] = v;
    xt[(size_t)p * Kp + l] = v;
  }
}

}  // namespace

hipError_t launch_learned_inputs(const double* W64, const float* feat, int P, int O, float* X, hipStream_t st) {
  hipLaunchKernelGGL(k_learned_inputs, dim3(P), dim3(128), 0, st, W64, feat, O, X);
  return hipGetLastError();
}

hipError_t launch_learned_start(const float* Y, int P, int Pp, int K, int Kp, const double* t_bar, double floor,
                                float* xe, hipStream_t st) {
  (void)Pp;
  hipLaunchKernelGGL(k_learned_start, dim3(P), dim3(128), 0, st, Y, K, Kp, t_bar, (float)floor, xe);
  return hipGetLastError();
}

hipError_t launch_pick_start(const double* F_warm, const double* F_uniform, const float* xe, int P, int Kp,
                             float* x, float* xt, int* n_warm, int* use_warm, hipStream_t st) {
  hipLaunchKernelGGL(k_pick_start, dim3(P), dim3(128), 0, st, F_warm, F_uniform, xe, Kp, x, xt, n_warm, use_warm);
  return hipGetLastError();
}

hipError_t launch_dose_rate(const double* dwell_xyz, const double* pt_xyz, const double* user_D,
                            const int* perm, int M, int K, int Mp, int Kp, double* D64,
                            hipStream_t st) {
  DoseArgs a{};
  a.dwell = dwell_xyz;
  a.pts = pt_xyz;
  a.user_D = user_D;
  a.perm = perm;
  a.M = M;
  a.K = K;
  a.Mp = Mp;
  a.Kp = Kp;
  a.D64 = D64;
  hipLaunchKernelGGL((k_dose_matrix<DOSE_D64>), dim3(Mp / 32), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_dose_setup(const double* dwell_xyz, const double* pt_xyz, const double* user_D,
                             const int* perm, int M, int K, int Mp, int Kp, int dtype, int row_begin,
                             int row_end, double prescription, double* D64, float* D32, void* Dlp, void* DTlp,
                             float* colscale, double* scratch, double* t_bar, hipStream_t st) {
  DoseArgs a{};
  a.dwell = dwell_xyz;
  a.pts = pt_xyz;
  a.user_D = user_D;
  a.perm = perm;
  a.M = M;
  a.K = K;
  a.Mp = Mp;
  a.Kp = Kp;
  a.r0 = row_begin;
  a.r1 = row_end;
  a.D64 = D64;
  a.D32 = D32;
  a.D16 = (uint16_t*)Dlp;
  a.DT16 = (uint16_t*)DTlp;
  a.rowsum = scratch;
  a.colmax = scratch + Mp;
  const dim3 grid(Mp / 32), block(256);
  if (dtype == GMCO_DTYPE_BF16) hipLaunchKernelGGL((k_dose_matrix<DOSE_BF16>), grid, block, 0, st, a);
  else if (dtype == GMCO_DTYPE_FP8) hipLaunchKernelGGL((k_dose_matrix<DOSE_FP8>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((k_dose_matrix<DOSE_F32>), grid, block, 0, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (dtype == GMCO_DTYPE_FP8) {
    hipLaunchKernelGGL(k_colscale, dim3((Kp + 63) / 64), dim3(1024), 0, st, a.colmax, Mp / 32, Kp, colscale);
    hipLaunchKernelGGL(k_cast_fp8, dim3(1024), dim3(256), 0, st, D32, (size_t)Mp * Kp / 4, Kp / 4, colscale,
                       (unsigned*)Dlp);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_start_time, dim3(1), dim3(1024), 0, st, a.rowsum, row_begin, row_end, prescription, t_bar);
  return hipGetLastError();
}

hipError_t launch_widen_fp8(const void* D8, const float* colscale, int Mp, int Kp, double* out,
                            hipStream_t st) {
  hipLaunchKernelGGL(k_widen_fp8, dim3(1024), dim3(256), 0, st, (const unsigned char*)D8,
                     colscale, Mp, Kp, out);
  return hipGetLastError();
}

hipError_t launch_init_plans(int P, int Pp, int K, int Kp, const double* t0, const double* t_bar,
                             const double* W, int G, int O, const int* gorg, const int* norm,
                             float* xt, float* x, float* wn, double* W64, PlanState* ps,
                             hipStream_t st) {
  hipLaunchKernelGGL(k_init_plans, dim3(Pp), dim3(128), 0, st, P, Pp, K, Kp, t0, t_bar, W, G, O,
                     gorg, norm, xt, x, wn, W64, ps);
  return hipGetLastError();
}

hipError_t launch_x_to_device(const double* x, int P, int Pp, int K, int Kp, float* xe, hipStream_t st) {
  hipLaunchKernelGGL((k_x_to_device<double>), dim3(Pp), dim3(128), 0, st, x, P, K, Kp, xe);
  return hipGetLastError();
}

hipError_t launch_x32_to_device(const float* x, int P, int Pp, int K, int Kp, float* xe, hipStream_t st) {
  hipLaunchKernelGGL((k_x_to_device<float>), dim3(Pp), dim3(128), 0, st, x, P, K, Kp, xe);
  return hipGetLastError();
}

}  // namespace gmco
