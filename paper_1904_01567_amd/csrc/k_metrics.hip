// Final-plan quantities in FP64: t = x^2, the dose of every point
// (eq. (dose)), eq. (obj) re-evaluated, and the DVH metrics of Sec. 2.3.1.
#include "gmco_internal.h"

namespace gmco {
namespace {

typedef double d4v __attribute__((ext_vector_type(4)));

// d64[p][i] = sum_l D64[i][l] x[p][l]^2 on the 16x16x4 FP64 matrix op, bound
// by its rate (67 TFLOP/s reached by a large library product on this chip),
// for few plans by the bytes of D64.  A wavefront computes 16 NA plans x 32
// points (A = plans, so that a store instruction writes whole 128-byte lines
// of four plans' rows); lane (q, n) reads 16 bytes of x and 32 of D64 per row
// and 16-dwell step, dwells 4 q .. 4 q + 3, i.e. matrix op s of the step
// contracts dwells 4 q + s.  Both operands go straight to registers, the next
// step's in flight: the plan tile's x is shared through the caches, D64 has no
// reuse within a workgroup.  Four wavefronts, 128 points; the plan tiles of a
// point range follow each other on one XCD, whose L2 then serves D64 to all but
// the first.  NA = 4 plan tiles per wavefront hold 64 accumulator registers (two
// wavefronts per SIMD, which the FP64 op needs for its rate); NA = 1, 2 leave
// out the empty tiles of batches up to 16 and 32 plans.  At 1,000 plans x 360
// dwells: 1.35 ms for 100,000 points (54 TFLOP/s) and 0.28 for 20,000, against 3.5
// and 0.7 ms with vector FMAs from LDS tiles.
template <int NA>
__global__ __launch_bounds__(256, 2) void k_dose64(const double* __restrict__ D64, const float* __restrict__ x,
                                                   int Mp, int K, int Kp, int P, int nptile, int nplan,
                                                   double* __restrict__ d64) {
  constexpr int NB = 2;
  const int tid = threadIdx.x;
  const int wave = tid >> 6, lane = tid & 63, q = lane >> 4, n = lane & 15;
  // workgroup -> (point tile, plan tile), point tiles round-robin over the XCDs
  const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
  const int pt = (local / nplan) * 8 + xcd;
  if (pt >= nptile) return;
  const int i0 = pt * 128 + wave * 32;
  const int p0 = (local % nplan) * 16 * NA;
  if (i0 >= Mp) return;  // (Mp is a multiple of 32)
  const double* __restrict__ drow[NB];
  const float* __restrict__ xrow[NA];
#pragma unroll
  for (int b = 0; b < NB; ++b) drow[b] = D64 + (size_t)(i0 + 16 * b + n) * Kp + 4 * q;
#pragma unroll
  for (int a = 0; a < NA; ++a) xrow[a] = x + (size_t)min(p0 + 16 * a + n, P - 1) * Kp + 4 * q;
  d4v acc[NA][NB];
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = d4v{0.0, 0.0, 0.0, 0.0};
  d4v dv[2][NB];
  float4 xv[2][NA];
  auto load = [&](int k, d4v (&dn)[NB], float4 (&xn)[NA]) {
#pragma unroll
    for (int b = 0; b < NB; ++b) dn[b] = *reinterpret_cast<const d4v*>(drow[b] + k);
#pragma unroll
    for (int a = 0; a < NA; ++a) xn[a] = *reinterpret_cast<const float4*>(xrow[a] + k);
    if (k + 16 > K) {  // padding dwells do not enter, whatever x holds there
#pragma unroll
      for (int a = 0; a < NA; ++a) {
        const int l = k + 4 * q;
        xn[a].x = l < K ? xn[a].x : 0.f;
        xn[a].y = l + 1 < K ? xn[a].y : 0.f;
        xn[a].z = l + 2 < K ? xn[a].z : 0.f;
        xn[a].w = l + 3 < K ? xn[a].w : 0.f;
      }
    }
  };
  auto step = [&](const d4v (&dn)[NB], const float4 (&xn)[NA]) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      double t[NA];
#pragma unroll
      for (int a = 0; a < NA; ++a) {
        const double xd = (double)(s == 0 ? xn[a].x : s == 1 ? xn[a].y : s == 2 ? xn[a].z : xn[a].w);
        t[a] = xd * xd;
      }
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(t[a], dn[b][s], acc[a][b], 0, 0, 0);
    }
  };
  // two register sets, a step ahead of its use (Kp is a multiple of 32, so the
  // last load of a pair of steps stays inside the row; D64 is zero past K)
  load(0, dv[0], xv[0]);
  for (int k = 0; k < K; k += 32) {
    load(k + 16, dv[1], xv[1]);
    step(dv[0], xv[0]);
    if (k + 32 < K) load(k + 32, dv[0], xv[0]);
    if (k + 16 < K) step(dv[1], xv[1]);
  }
  // accumulator register r: plan q + 4 r, point n
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int p = p0 + 16 * a + q + 4 * r;
      if (p >= P) continue;
#pragma unroll
      for (int b = 0; b < NB; ++b) d64[(size_t)p * Mp + i0 + 16 * b + n] = acc[a][b][r];
    }
}

// k-th largest of the keys (bit patterns of non-negative doubles order like
// their values), radix select over 8-bit digits from the most significant.
struct SelectState {
  unsigned long long prefix;
  unsigned long long mask;
  int k;
};

__device__ inline double wave_add(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

constexpr int kMT = 512;        // threads of a (plan, organ) workgroup
constexpr int kBins = 4096;     // bins of the dose histogram
constexpr int kCand = 1024;     // doses of the selected bin that fit LDS
// Bin of a dose's bit pattern: 256 bins per octave over 2^-4 .. 2^12 Gy, the
// doses below and above in the first and last bin.  Monotone in the pattern.
__device__ inline int dose_bin(unsigned long long key) {
  const int b = (int)(key >> 44) - ((1023 - 4) << 8);
  return min(max(b, 0), kBins - 1);
}

// One workgroup per (plan, organ): the organ's points of one point set
// (MetricsArgs).  The individual objective f_j = (1/N_j) sum f_i takes each
// point's own group parameters (surface and volume rows of one organ share the
// organ's N_j); the DVH metrics follow the definitions of Sec. 2.3.1 (V_x
// counts d >= x % Rx; D_x is the k-th hottest dose, k = max(1, ceil(x N / 100)).
// Bound by the reads of the doses, so there are two: the first adds the
// objective, counts V_x and fills a histogram of the doses' bit patterns, whose
// counts from the top give the bins of D10 and D90; the second collects the
// doses of these two bins, and each is ranked among its bin exactly.  Bins of
// more than kCand doses (many equal doses) go through a radix select over the
// FP64 bit patterns, eight reads, instead.  1,000 plans with 100,000 points:
// 0.25 ms, against 1.8 with the radix select for all (nine reads, its first
// digits' counts contended by every lane).
__global__ __launch_bounds__(kMT) void k_metrics_group(MetricsArgs a) {
  constexpr int NW = kMT / 64, U = 8;
  __shared__ unsigned int hist[kBins];
  __shared__ double cand[2][kCand];
  __shared__ double red[3][NW];
  __shared__ double prm[kGmax][4];
  __shared__ unsigned int wsum[NW];
  __shared__ int bin[2], rank[2], inbin[2], ncand[2];
  __shared__ SelectState sel[2];
  const int p = blockIdx.x;
  const int j = blockIdx.y;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  if (p >= a.P) return;
  gmco_plan_metrics* m = a.out + p;
  if (j >= a.O) {
    if (tid == 0 && j < kGmax) {
      if (a.objective) m->f_organ[j] = 0.0;
      if (a.dvh) {
        m->V100_pct[j] = 0.0;
        m->V75_cc[j] = 0.0;
        m->D10_pct[j] = 0.0;
        m->D90_pct[j] = 0.0;
      }
    }
    return;
  }
  const int N = a.cnt[j];
  const int o0 = a.off[j];
  const double* __restrict__ d = a.d64 + (size_t)p * a.ld + o0;
  const double thr100 = a.rx, thr75 = 0.75 * a.rx;

  for (int i = tid; i < kBins; i += kMT) hist[i] = 0u;
  if (tid < kGmax * 4) (&prm[0][0])[tid] = a.gparams[tid];
  if (tid < 2) ncand[tid] = 0;
  __syncthreads();
  double fs = 0.0;
  int c100 = 0, c75 = 0;
  for (int i0 = tid; i0 < N; i0 += U * kMT) {
    double v[U];
    int g[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = min(i0 + u * kMT, N - 1);
      v[u] = d[i];
      g[u] = a.objective ? a.grp[o0 + i] : 0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (i0 + u * kMT >= N) break;
      if (a.objective) {
        const double wmin = prm[g[u]][0], dmin = prm[g[u]][1], dmax = prm[g[u]][2], wmax = prm[g[u]][3];
        if (v[u] < dmin) fs += wmin * ((dmin - v[u]) * (dmin - v[u]));
        else if (v[u] > dmax) fs += wmax * ((v[u] - dmax) * (v[u] - dmax));
      }
      c100 += v[u] >= thr100 ? 1 : 0;
      c75 += v[u] >= thr75 ? 1 : 0;
      if (a.dvh) atomicAdd(&hist[dose_bin((unsigned long long)__double_as_longlong(v[u]))], 1u);
    }
  }
  {
    const double s0 = wave_add(fs), s1 = wave_add((double)c100), s2 = wave_add((double)c75);
    if (lane == 0) {
      red[0][wave] = s0;
      red[1][wave] = s1;
      red[2][wave] = s2;
    }
  }
  __syncthreads();
  double tot[3];
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    tot[t] = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) tot[t] += red[t][w];
  }
  if (a.objective && tid == 0) m->f_organ[j] = tot[0] / (N > 0 ? (double)N : 1.0);
  if (!a.dvh) return;
  const double n = N > 0 ? (double)N : 1.0;
  if (tid == 0) {
    m->V100_pct[j] = 100.0 * (tot[1] / n);
    m->V75_cc[j] = (a.volume_cc ? a.volume_cc[j] : 0.0) * (tot[2] / n);
    if (N == 0) m->D10_pct[j] = m->D90_pct[j] = 0.0;
  }
  if (N == 0) return;

  // D10 / D90: k = max(1, ceil(x N / 100)) in integers.  Counts from the top:
  // thread t takes bins kBins - 1 - 8 t downwards.
  const int k2[2] = {max(1, (int)((10ll * N + 99) / 100)), max(1, (int)((90ll * N + 99) / 100))};
  constexpr int PB = kBins / kMT;
  unsigned int own = 0;
#pragma unroll
  for (int u = 0; u < PB; ++u) own += hist[kBins - 1 - PB * tid - u];
  unsigned int incl = own;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned int up = __shfl_up(incl, o);
    if (lane >= o) incl += up;
  }
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  unsigned int above = incl - own;
  for (int w = 0; w < wave; ++w) above += wsum[w];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    if (above < (unsigned)k2[t] && (unsigned)k2[t] <= above + own) {
      unsigned int c = above;
      for (int u = 0; u < PB; ++u) {
        const unsigned int h = hist[kBins - 1 - PB * tid - u];
        if ((unsigned)k2[t] <= c + h) {
          bin[t] = kBins - 1 - PB * tid - u;
          rank[t] = k2[t] - (int)c;
          inbin[t] = (int)h;
          break;
        }
        c += h;
      }
    }
  }
  __syncthreads();
  const int b0 = bin[0], b1 = bin[1];
  if (inbin[0] <= kCand && inbin[1] <= kCand) {
    for (int i0 = tid; i0 < N; i0 += U * kMT) {
      double v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = d[min(i0 + u * kMT, N - 1)];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (i0 + u * kMT >= N) break;
        const int b = dose_bin((unsigned long long)__double_as_longlong(v[u]));
        if (b == b0) cand[0][atomicAdd(&ncand[0], 1)] = v[u];
        if (b == b1) cand[1][atomicAdd(&ncand[1], 1)] = v[u];
      }
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int c = inbin[t];
      for (int i = tid; i < c; i += kMT) {
        const unsigned long long key = (unsigned long long)__double_as_longlong(cand[t][i]);
        int gt = 0, ge = 0;
        for (int e = 0; e < c; ++e) {
          const unsigned long long o = (unsigned long long)__double_as_longlong(cand[t][e]);
          gt += o > key ? 1 : 0;
          ge += o >= key ? 1 : 0;
        }
        if (gt < rank[t] && rank[t] <= ge) (t == 0 ? m->D10_pct : m->D90_pct)[j] = 100.0 * cand[t][i] / a.rx;
      }
    }
    return;
  }

  // many equal doses: radix select
  unsigned int* h10 = hist;
  unsigned int* h90 = hist + 256;
  if (tid < 2) {
    sel[tid].prefix = 0ull;
    sel[tid].mask = 0ull;
    sel[tid].k = k2[tid];
  }
  __syncthreads();
  for (int shift = 56; shift >= 0; shift -= 8) {
    hist[tid] = 0u;  // (512 threads: both histograms)
    __syncthreads();
    const unsigned long long pf0 = sel[0].prefix, mk0 = sel[0].mask;
    const unsigned long long pf1 = sel[1].prefix, mk1 = sel[1].mask;
    for (int i = tid; i < N; i += kMT) {
      const unsigned long long key = (unsigned long long)__double_as_longlong(d[i]);
      const unsigned dig = (unsigned)((key >> shift) & 0xffull);
      if ((key & mk0) == pf0) atomicAdd(&h10[dig], 1u);
      if ((key & mk1) == pf1) atomicAdd(&h90[dig], 1u);
    }
    __syncthreads();
    if (tid < 2) {
      unsigned int* h = tid == 0 ? h10 : h90;
      SelectState& s = sel[tid];
      int k = s.k;
      int dsel = 0;
      for (int dg = 255; dg >= 0; --dg) {
        const int c = (int)h[dg];
        if (k <= c) {
          dsel = dg;
          break;
        }
        k -= c;
      }
      s.k = k;
      s.prefix |= ((unsigned long long)dsel) << shift;
      s.mask |= 0xffull << shift;
    }
    __syncthreads();
  }
  if (tid == 0) {
    m->D10_pct[j] = 100.0 * __longlong_as_double((long long)sel[0].prefix) / a.rx;
    m->D90_pct[j] = 100.0 * __longlong_as_double((long long)sel[1].prefix) / a.rx;
  }
}

__global__ void k_metrics_final(const double* __restrict__ W64, const PlanState* __restrict__ ps,
                                int P, int O, gmco_plan_metrics* __restrict__ out) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= P) return;
  gmco_plan_metrics* m = out + p;
  double F = 0.0;
  for (int j = 0; j < O; ++j) F += W64[(size_t)p * kGmax + j] * m->f_organ[j];
  m->F64 = F;
  m->F_run = ps[p].F;
  m->iterations = ps[p].iter;
  m->evaluations = ps[p].nevals;
  m->status = ps[p].status == ST_INIT ? ST_RUNNING : ps[p].status;
  m->reserved = 0;
}

// Per plan, RTOG 0924 class (Sec. 2.3.1: 2 = RTOG+ valid, 1 = RTOG valid, 0 =
// invalid) and dominance: plan p is dominated when another plan is at least as
// good in every individual objective and strictly better in one (Sec. 2.2.4).
// A workgroup takes kParetoP plans and runs every plan q past them, one per
// thread and step: a load of q's objectives serves kParetoP comparisons.  (One
// thread per plan running through all others by itself took 627 us at 1,000
// plans, a dependent load each; this takes 15, the classes included.)
constexpr int kParetoP = 16;
__global__ __launch_bounds__(256) void k_classify_pareto(const gmco_plan_metrics* __restrict__ m, int P, int G,
                                                         gmco_select_opts o, int* __restrict__ cls,
                                                         int* __restrict__ meets_tu, int* __restrict__ nd) {
  __shared__ double f[kParetoP][kGmax];
  __shared__ unsigned int dominated;
  const int p0 = blockIdx.x * kParetoP;
  const int tid = threadIdx.x;
  if (tid == 0) dominated = 0u;
  for (int i = tid; i < kParetoP * G; i += 256) f[i / G][i % G] = m[min(p0 + i / G, P - 1)].f_organ[i % G];
  __syncthreads();
  unsigned int dom = 0;
  for (int q = tid; q < P; q += 256) {
    unsigned int le = ~0u, lt = 0u;
    for (int j = 0; j < G; ++j) {
      const double a = m[q].f_organ[j];
#pragma unroll
      for (int i = 0; i < kParetoP; ++i) {
        const double b = f[i][j];
        if (!(a <= b)) le &= ~(1u << i);
        if (a < b) lt |= 1u << i;
      }
    }
    if (q >= p0 && q < p0 + kParetoP) lt &= ~(1u << (q - p0));
    dom |= le & lt;
  }
  if (dom) atomicOr(&dominated, dom);
  __syncthreads();
  const int p = p0 + tid;
  if (tid >= kParetoP || p >= P) return;
  nd[p] = (dominated >> tid) & 1u ? 0 : 1;
  const double v100 = m[p].V100_pct[o.target];
  const bool ok_t = v100 >= o.v100_min;
  const bool ok_u = m[p].D10_pct[o.urethra] < o.urethra_d10_max;
  const bool ok_b = m[p].V75_cc[o.bladder] < o.bladder_v75_max;
  const bool ok_r = m[p].V75_cc[o.rectum] < o.rectum_v75_max;
  cls[p] = (ok_t && ok_u && ok_b && ok_r) ? (v100 >= o.v100_plus ? 2 : 1) : 0;
  meets_tu[p] = (ok_t && ok_u) ? 1 : 0;
}

// Selection (Sec. 2.4): RTOG+ over RTOG over invalid; among valid plans the
// highest target V100; among invalid plans the lowest bladder + rectum V75
// among those meeting the target and urethra criteria (all invalid plans if
// none does); ties to the lowest index.  One workgroup.
__global__ __launch_bounds__(1024) void k_select(const gmco_plan_metrics* __restrict__ m,
                                                 const int* __restrict__ cls,
                                                 const int* __restrict__ meets_tu, const int* __restrict__ nd,
                                                 int P, gmco_select_opts o, int* __restrict__ out) {
  __shared__ int s_i[1024];
  __shared__ double s_k[1024];
  const int t = threadIdx.x;
  // best class and whether an invalid plan meets target and urethra
  int bc = 0, tu = 0, nnd = 0;
  for (int p = t; p < P; p += blockDim.x) {
    bc = max(bc, cls[p]);
    tu |= (cls[p] == 0 && meets_tu[p]) ? 1 : 0;
    nnd += nd[p];
  }
  s_i[t] = bc;
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if (t < w) s_i[t] = max(s_i[t], s_i[t + w]);
    __syncthreads();
  }
  const int best_class = s_i[0];
  __syncthreads();
  s_i[t] = tu;
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if (t < w) s_i[t] = s_i[t] | s_i[t + w];
    __syncthreads();
  }
  const int any_tu = s_i[0];
  __syncthreads();
  s_i[t] = nnd;
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if (t < w) s_i[t] += s_i[t + w];
    __syncthreads();
  }
  const int n_nd = s_i[0];
  __syncthreads();
  // smallest key wins, ties to the lowest index
  int bi = -1;
  double bk = 0.0;
  for (int p = t; p < P; p += blockDim.x) {
    if (cls[p] != best_class) continue;
    if (best_class == 0 && any_tu && !meets_tu[p]) continue;
    const double key = best_class > 0 ? -m[p].V100_pct[o.target]
                                       : m[p].V75_cc[o.bladder] + m[p].V75_cc[o.rectum];
    if (bi < 0 || key < bk) {
      bi = p;
      bk = key;
    }
  }
  s_i[t] = bi;
  s_k[t] = bk;
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if (t < w) {
      const int i2 = s_i[t + w];
      const double k2 = s_k[t + w];
      if (i2 >= 0 && (s_i[t] < 0 || k2 < s_k[t] || (k2 == s_k[t] && i2 < s_i[t]))) {
        s_i[t] = i2;
        s_k[t] = k2;
      }
    }
    __syncthreads();
  }
  if (t == 0) {
    out[0] = s_i[0];
    out[1] = n_nd;
  }
}

}  // namespace

hipError_t launch_select(const gmco_plan_metrics* m, int P, int G, const gmco_select_opts& o, int* cls,
                         int* meets_tu, int* nd, int* out, hipStream_t st) {
  hipLaunchKernelGGL(k_classify_pareto, dim3((P + kParetoP - 1) / kParetoP), dim3(256), 0, st, m, P, G, o, cls,
                     meets_tu, nd);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_select, dim3(1), dim3(1024), 0, st, m, cls, meets_tu, nd, P, o, out);
  return hipGetLastError();
}

hipError_t launch_dose64(const double* D64, const float* x, int Mp, int K, int Kp, int P, double* d64,
                         hipStream_t st) {
  const int na = P <= 16 ? 1 : P <= 32 ? 2 : 4;
  const int nptile = (Mp + 127) / 128, nplan = (P + 16 * na - 1) / (16 * na);
  const dim3 grid((unsigned)((nptile + 7) / 8 * 8) * nplan);
  if (na == 1)
    hipLaunchKernelGGL((k_dose64<1>), grid, dim3(256), 0, st, D64, x, Mp, K, Kp, P, nptile, nplan, d64);
  else if (na == 2)
    hipLaunchKernelGGL((k_dose64<2>), grid, dim3(256), 0, st, D64, x, Mp, K, Kp, P, nptile, nplan, d64);
  else
    hipLaunchKernelGGL((k_dose64<4>), grid, dim3(256), 0, st, D64, x, Mp, K, Kp, P, nptile, nplan, d64);
  return hipGetLastError();
}

hipError_t launch_metrics(const MetricsArgs& m, hipStream_t st) {
  if (m.P < 1) return hipSuccess;
  hipLaunchKernelGGL(k_metrics_group, dim3(m.P, kGmax), dim3(kMT), 0, st, m);
  return hipGetLastError();
}

hipError_t launch_metrics_final(const MetricsArgs& m, hipStream_t st) {
  if (m.P < 1) return hipSuccess;
  hipLaunchKernelGGL(k_metrics_final, dim3((m.P + 127) / 128), dim3(128), 0, st, m.W64, m.ps, m.P,
                     m.O, m.out);
  return hipGetLastError();
}

}  // namespace gmco
