// Learned warm start: a fully connected ReLU network trained on plans the
// method itself produced, and the case features it reads.
//
// Every product runs on v_mfma_f32_16x16x32_bf16 (BF16 operands rounded from
// FP32 activations and weights, FP32 accumulation); losses, gradients and the
// Adam moments are FP32.  Parameter layout: for each layer W (n_out x n_in,
// row-major) followed by b (n_out).
#include <algorithm>
#include <cstring>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "gmco_internal.h"

namespace gmco {
namespace {

typedef float f4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));

// The network's products C[i][j] = sum_k A[i][k] B[k][j] on 16x16x32 BF16
// matrix ops, in the three forms of a training step:
//   FWD   act' = relu?(act W^T + b): A and B contiguous in k;
//   DACT  dact = (G W) masked by act > 0: A contiguous in k, B in j;
//   DW    dW = G^T act, contraction over the batch: A contiguous in i, B in j.
// A workgroup of four wavefronts (2 x 2) computes a T x T tile.  Slices of 64
// k are read along the contiguous dimension into registers, four slices ahead
// (two with T = 64), and staged in LDS as BF16, 16 bytes a store (two buffers,
// one barrier per slice).  The sizes of this network leave every product bound
// by latency: few tiles, each a chain of slices.  So T = 32 unless 64 x 64 tiles
// already fill the chip twice (kGemmWide), all weight gradients of a step are
// one launch, and what the epilogue reads is loaded before the chain.  The
// contraction runs in ascending steps of 32 in every form and tile, so the
// tile does not change a bit of the result.
// Measured (batch 1,024, layers 68-256-256-256-360): 73 us per product with
// 64 x 64 tiles, strided scalar loads and no prefetch, 11 products a step, 1,785
// us.  With 32 x 32 tiles, two slices ahead, 2-byte stores and the bias sums' adds
// each waiting for LDS: 8.6 (forward), 12.4 (with the loss), 6.5 (activations) and
// 21.3 us (weights), a step 87.  Now 4.2, 7.2, 5.3 and 16.4, a step 59.  (Giving
// each XCD a rectangle of the weight gradients' tiles, which halves what its L2
// reads, changes nothing: 16.2.)
enum { GEMM_FWD = 0, GEMM_FWD_MSE = 1, GEMM_DACT = 2, GEMM_DW = 3, GEMM_DW_ADAM = 4 };

struct AdamArgs {
  float lr, b1, b2, eps, c1, c2;
};

struct GemmArgs {
  const float* A;
  const float* B;
  const int* rows;     // FWD: row i of A is rows[i] (NULL: itself), and
  float* gathered;     // these rows are written here (M x K)
  float* C;
  const float* bias;   // FWD: per column j
  const float* act;    // DACT: activations that mask C (same shape)
  const float* y;      // FWD_MSE: targets, row i at yrows[i]
  const int* yrows;
  double* loss;        // FWD_MSE: squared error of each tile
  float scale;         // FWD_MSE: 2 / (M N)
  float *p, *m, *v;    // DW_ADAM: parameters and moments, C's layout
  int lda, ldb;        // elements between rows of A and B as stored
  int M, N, K;
  int relu;
};

constexpr int kGemmWide = 512;  // 64 x 64 tiles from this many workgroups (two per compute unit)
constexpr int kKS = 64;         // k per slice
constexpr int kTS = kKS + 8;    // LDS row stride: 144 B, 16-byte aligned operand reads

// Adam's update from the gradient gi; the order of the fused operations is
// written out so that every caller rounds alike.
__device__ inline void adam_update(float gi, float& p, float& m, float& v, const AdamArgs& a) {
  m = fmaf(1.f - a.b1, gi, a.b1 * m);
  v = fmaf(gi, (1.f - a.b2) * gi, a.b2 * v);
  p -= a.lr * (m / a.c1) / (sqrtf(v / a.c2) + a.eps);
}

// A thread's share of the slices of an operand, T rows (i or j) x 64 k: NU
// groups of 8 consecutive k of one row, so that a group is one 16-byte store to
// LDS.  KC: the stored rows are this operand's rows, contiguous in k (row r at
// rows[r] if given), by 16-byte loads if WIDE (rows of whole, aligned float4);
// otherwise the stored rows are k, contiguous in the operand's rows: a scalar
// address for each and one 32-bit offset per thread.  Places past the matrix
// read its last row or column: a load inside a branch that issues none on its
// other side would make every wait for an older one a wait for all (the count
// of those in flight is then unknown to the compiler).  Past K they are staged
// as zero; past the rows they reach only results that are not stored.
template <int T, bool KC, bool WIDE>
struct Operand {
  static constexpr int NU = T * kKS / 8 / 256;
  const float* src;
  const float* base[NU];  // KC: the row
  unsigned off[NU];       // otherwise: bytes from the slice's first stored row
  int r0, R, K, ld;

  __device__ static int row(int u) { return KC ? (threadIdx.x + 256 * u) / 8 : (threadIdx.x + 256 * u) % T; }
  __device__ static int kgrp(int u) { return KC ? (threadIdx.x + 256 * u) % 8 : (threadIdx.x + 256 * u) / T; }

  __device__ Operand(const float* src_, const int* rows, int ld_, int r0_, int R_, int K_)
      : src(src_), r0(r0_), R(R_), K(K_), ld(ld_) {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int r = min(r0 + row(u), R - 1);
      if constexpr (KC) base[u] = src + (size_t)(rows ? rows[r] : r) * ld;
      else off[u] = 4u * (8u * kgrp(u) * ld + (r - r0));
    }
  }
  // INSIDE: the slice ends at or before K
  template <bool INSIDE>
  __device__ void load(int k0, float (&v)[8 * NU]) const {
    if constexpr (KC) {
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const int k = k0 + 8 * kgrp(u);
        if constexpr (WIDE) {
          const f4v lo = *reinterpret_cast<const f4v*>(base[u] + min(k, K - 4));
          const f4v hi = *reinterpret_cast<const f4v*>(base[u] + min(k + 4, K - 4));
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            v[8 * u + e] = lo[e];
            v[8 * u + 4 + e] = hi[e];
          }
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) v[8 * u + e] = base[u][min(k + e, K - 1)];
        }
      }
    } else if constexpr (INSIDE) {
      const char* s0 = reinterpret_cast<const char*>(src + (size_t)k0 * ld + r0);
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int e = 0; e < 8; ++e)
          v[8 * u + e] = *reinterpret_cast<const float*>(s0 + (size_t)(4 * e) * ld + off[u]);
    } else {
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int e = 0; e < 8; ++e)
          v[8 * u + e] =
              src[(size_t)min(k0 + 8 * kgrp(u) + e, K - 1) * ld + min(r0 + row(u), R - 1)];
    }
  }
  // LAST: the slice may end past K
  template <bool LAST>
  __device__ void stage(__bf16* dst, int k0, const float (&v)[8 * NU]) const {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      bf8v w;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float x = v[8 * u + e];
        if (LAST && k0 + 8 * kgrp(u) + e >= K) x = 0.f;
        w[e] = (__bf16)x;
      }
      *reinterpret_cast<bf8v*>(&dst[row(u) * kTS + 8 * kgrp(u)]) = w;
    }
  }
};

template <int T, int FORM, bool WIDE>
__device__ inline void gemm_tile(const GemmArgs& g, int bi, int bj, const AdamArgs& ad) {
  constexpr bool AK = FORM <= GEMM_DACT, BK = FORM <= GEMM_FWD_MSE;
  constexpr int NL = 8 * Operand<T, true, false>::NU;
  constexpr int NP = T == 32 ? 4 : 2;  // slices in flight (even: two LDS buffers in turn)
  enum { NONE, CLAMPED, INSIDE };      // what a step loads: nothing, a slice that may end past K, one that does not
  constexpr int S = T / 32;  // 16-wide sub-tiles per wavefront and side
  __shared__ __attribute__((aligned(16))) __bf16 sA[2][T * kTS];
  __shared__ __attribute__((aligned(16))) __bf16 sB[2][T * kTS];
  __shared__ double sL[4];
  const int tid = threadIdx.x;
  const int wave = tid >> 6, lane = tid & 63, q = lane >> 4, n = lane & 15;
  const int i0 = bi * T, j0 = bj * T;
  const int wr = (wave >> 1) * (T / 2), wc = (wave & 1) * (T / 2);
  f4v acc[S][S];
#pragma unroll
  for (int a = 0; a < S; ++a)
#pragma unroll
    for (int b = 0; b < S; ++b) acc[a][b] = f4v{0.f, 0.f, 0.f, 0.f};
  const Operand<T, BK, WIDE> opB(g.B, nullptr, g.ldb, j0, g.N, g.K);
  const Operand<T, AK, WIDE> opA(g.A, FORM <= GEMM_FWD_MSE ? g.rows : nullptr, g.lda, i0, g.M, g.K);
  float ra[NP][NL], rb[NP][NL];
  const int ns = (g.K + kKS - 1) / kKS;
#pragma unroll
  for (int u = 0; u < NP; ++u) {
    opB.template load<false>(u * kKS, rb[u]);
    opA.template load<false>(u * kKS, ra[u]);
  }
  // element e = (a, b, r) of the tile: row and column of accumulator register r
  auto row = [&](int e) { return i0 + wr + 16 * (e / (4 * S)) + 4 * q + e % 4; };
  auto col = [&](int e) { return j0 + wc + 16 * (e / 4 % S) + n; };
  constexpr int NE = 4 * S * S;
  float e0[NE], e1[NE], e2[NE];  // what the epilogue reads, all loads in flight together
  auto epilogue_loads = [&]() {
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const int i = min(row(e), g.M - 1), j = min(col(e), g.N - 1);
      const size_t at = (size_t)i * g.N + j;
      if constexpr (FORM <= GEMM_FWD_MSE) e0[e] = g.bias[j];
      if constexpr (FORM == GEMM_FWD_MSE) e1[e] = g.y[(size_t)(g.yrows ? g.yrows[i] : i) * g.N + j];
      if constexpr (FORM == GEMM_DACT) e0[e] = g.act[at];
      if constexpr (FORM == GEMM_DW_ADAM) {
        e0[e] = g.p[at];
        e1[e] = g.m[at];
        e2[e] = g.v[at];
      }
    }
  };
  if constexpr (T == 32) epilogue_loads();  // (64 x 64: the registers are the accumulators')
  auto step = [&](int s, __bf16* cA, __bf16* cB, float (&va)[NL], float (&vb)[NL], auto next) {
    __builtin_amdgcn_sched_barrier(0);  // (no wait for a later slice moves up)
    opA.template stage<next() == NONE>(cA, s * kKS, va);
    opB.template stage<next() == NONE>(cB, s * kKS, vb);
    if constexpr (FORM <= GEMM_FWD_MSE) {
      // the gathered rows, for the weight gradient (whose contraction over
      // them would otherwise wait for each slice's row indices)
      if (g.rows && bj == 0) {
#pragma unroll
        for (int e = 0; e < NL; ++e) {
          const int i = i0 + opA.row(e / 8), k = s * kKS + 8 * opA.kgrp(e / 8) + e % 8;
          if (i < g.M && k < g.K) g.gathered[(size_t)i * g.K + k] = va[e];
        }
      }
    }
    if constexpr (next() != NONE) {
      opB.template load<next() == INSIDE>((s + NP) * kKS, vb);
      opA.template load<next() == INSIDE>((s + NP) * kKS, va);
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < kKS / 32; ++h) {
      if (next() == NONE && s * kKS + 32 * h >= g.K) break;
      bf8v af[S], bfr[S];
#pragma unroll
      for (int a = 0; a < S; ++a) {
        af[a] = *reinterpret_cast<const bf8v*>(&cA[(wr + 16 * a + n) * kTS + 32 * h + 8 * q]);
        bfr[a] = *reinterpret_cast<const bf8v*>(&cB[(wc + 16 * a + n) * kTS + 32 * h + 8 * q]);
      }
#pragma unroll
      for (int a = 0; a < S; ++a)
#pragma unroll
        for (int b = 0; b < S; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[a], bfr[b], acc[a][b], 0, 0, 0);
    }
  };
  auto steps = [&](int s, auto next) {
#pragma unroll
    for (int u = 0; u < NP; ++u)
      if (next() != NONE || s + u < ns) step(s + u, sA[u & 1], sB[u & 1], ra[u], rb[u], next);
  };
  int s = 0;
  for (; (s + 2 * NP) * kKS <= g.K; s += NP) steps(s, std::integral_constant<int, INSIDE>());
  if (s + NP < ns) {
    steps(s, std::integral_constant<int, CLAMPED>());
    s += NP;
  }
  steps(s, std::integral_constant<int, NONE>());
  if constexpr (T != 32) epilogue_loads();
  double sq = 0.0;
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    const int i = row(e), j = col(e);
    if (i >= g.M || j >= g.N) continue;
    const size_t at = (size_t)i * g.N + j;
    float v = acc[e / (4 * S)][e / 4 % S][e % 4];
    if constexpr (FORM <= GEMM_FWD_MSE) v += e0[e];
    if constexpr (FORM == GEMM_FWD) {
      if (g.relu) v = fmaxf(v, 0.f);
    }
    if constexpr (FORM == GEMM_FWD_MSE) {
      // dL/dout for L = mean((out - y)^2)
      const float d = v - e1[e];
      sq += (double)d * (double)d;
      v = g.scale * d;
    }
    if constexpr (FORM == GEMM_DACT) {
      if (!(e0[e] > 0.f)) v = 0.f;
    }
    if constexpr (FORM == GEMM_DW_ADAM) {
      adam_update(v, e0[e], e1[e], e2[e], ad);
      g.p[at] = e0[e];
      g.m[at] = e1[e];
      g.v[at] = e2[e];
    } else {
      g.C[at] = v;
    }
  }
  if constexpr (FORM == GEMM_FWD_MSE) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) sq += __shfl_xor(sq, o);
    if (lane == 0) sL[wave] = sq;
    __syncthreads();
    if (tid == 0) g.loss[(size_t)bi * gridDim.y + bj] = (sL[0] + sL[1]) + (sL[2] + sL[3]);
  }
}

template <int T, int FORM, bool WIDE>
__global__ __launch_bounds__(256, 2) void k_gemm(GemmArgs g) {
  gemm_tile<T, FORM, WIDE>(g, blockIdx.x, blockIdx.y, AdamArgs{});
}

// Bias gradient db[j] = sum_i g[i][j] of 64 columns, in row order: chunks of
// 64 rows through registers (the next four in flight) into LDS (two buffers),
// added by one wavefront, whose reads of a chunk are all issued before its adds.
__device__ __forceinline__ float bias_sum(const float* __restrict__ G, int B, int N, int j0) {
  constexpr int R = 16, NP = 4;
  __shared__ float sG[2][4 * R][64];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int j = min(j0 + lane, N - 1);
  float v[NP][R];
  auto load = [&](int b, float (&w)[R]) {
#pragma unroll
    for (int u = 0; u < R; ++u) w[u] = G[(size_t)min(b + wave * R + u, B - 1) * N + j];
  };
  float s = 0.f;
#pragma unroll
  for (int c = 0; c < NP; ++c) load(4 * R * c, v[c]);
  auto step = [&](int b, float (&w)[R], float (*sg)[64], auto more) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < R; ++u) sg[wave * R + u][lane] = w[u];
    if constexpr (more()) load(b + 4 * R * NP, w);
    __syncthreads();
    if (wave == 0) {
      float w64[4 * R];
#pragma unroll
      for (int i = 0; i < 4 * R; ++i) w64[i] = sg[i][lane];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 4 * R; ++i)
        if (more() || b + i < B) s += w64[i];
    }
  };
  int b = 0;  // (the last 1 to NP chunks apart: their steps load nothing)
  for (; b + 4 * R * NP < B; b += 4 * R * NP) {
#pragma unroll
    for (int c = 0; c < NP; ++c) step(b + 4 * R * c, v[c], sG[c & 1], std::true_type());
  }
#pragma unroll
  for (int c = 0; c < NP; ++c)
    if (b + 4 * R * c < B) step(b + 4 * R * c, v[c], sG[c & 1], std::false_type());
  return s;
}

// Weight and bias gradients of up to kDwLayers layers in one launch: layer l's
// tiles are workgroups first[l] .. first[l + 1] - 1, its bias columns the last
// ceil(out / 64) of them.  ADAM: the parameters are updated in place of
// storing the gradient (nothing later in the step reads them).
constexpr int kDwLayers = 6;
struct DwArgs {
  GemmArgs g[kDwLayers];
  float* db[kDwLayers];  // bias gradient; ADAM: bias parameters, with their moments
  float* dbm[kDwLayers];
  float* dbv[kDwLayers];
  int first[kDwLayers + 1];
  int n;
  AdamArgs ad;
};

template <int T, bool ADAM>
__global__ __launch_bounds__(256, 2) void k_dw(DwArgs a) {
  int l = 0;
  while (l + 1 < a.n && (int)blockIdx.x >= a.first[l + 1]) ++l;
  const GemmArgs& g = a.g[l];
  const int t = blockIdx.x - a.first[l];
  const int tj = (g.N + T - 1) / T, tiles = tj * ((g.M + T - 1) / T);
  if (t < tiles) {
    gemm_tile<T, ADAM ? GEMM_DW_ADAM : GEMM_DW, false>(g, t / tj, t % tj, a.ad);
  } else {
    const int j0 = (t - tiles) * 64;
    const int j = j0 + (int)threadIdx.x;
    const bool own = threadIdx.x < 64 && j < g.M;
    float p = 0.f, m = 0.f, v = 0.f;
    if (ADAM && own) {
      p = a.db[l][j];
      m = a.dbm[l][j];
      v = a.dbv[l][j];
    }
    const float s = bias_sum(g.A, g.K, g.M, j0);
    if (!own) return;
    if constexpr (ADAM) {
      adam_update(s, p, m, v, a.ad);
      a.db[l][j] = p;
      a.dbm[l][j] = m;
      a.dbv[l][j] = v;
    } else {
      a.db[l][j] = s;
    }
  }
}

// Mean squared error of step blockIdx.x from its tiles' sums, in a fixed order.
__global__ __launch_bounds__(256) void k_sum_loss(const double* __restrict__ tile_loss, int n, double count,
                                                  double* __restrict__ out) {
  __shared__ double red[256];
  const double* src = tile_loss + (size_t)blockIdx.x * n;
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) s += src[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = blockDim.x / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[blockIdx.x] = red[0] / count;
}

// Case features: for dwell l and structure j the distance to the nearest
// point of j, binned in 16 bins of 0.25 cm (the last open-ended), divided by
// the dwell count.  (dx^2 + dy^2) + dz^2 without fused operations.
__global__ void k_features(const double* __restrict__ dwell, const double* __restrict__ pts,
                           const int* __restrict__ perm, const int* __restrict__ goff,
                           const int* __restrict__ gcnt, int K, unsigned* __restrict__ hist) {
  const int l = blockIdx.x, j = blockIdx.y;
  if (l >= K) return;  // (whole workgroup)
  __shared__ double red[256];
  double best = 1e300;
  const double qx = dwell[3 * l], qy = dwell[3 * l + 1], qz = dwell[3 * l + 2];
  for (int i = threadIdx.x; i < gcnt[j]; i += blockDim.x) {
    const int src = perm[goff[j] + i];
    const double dx = __dsub_rn(pts[3 * src], qx), dy = __dsub_rn(pts[3 * src + 1], qy);
    const double dz = __dsub_rn(pts[3 * src + 2], qz);
    const double r2 = __dadd_rn(__dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy)), __dmul_rn(dz, dz));
    best = fmin(best, r2);
  }
  red[threadIdx.x] = best;
  __syncthreads();
  for (int o = blockDim.x / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] = fmin(red[threadIdx.x], red[threadIdx.x + o]);
    __syncthreads();
  }
  if (threadIdx.x == 0 && gcnt[j] > 0) {
    const double r = sqrt(red[0]);
    int b = (int)floor(r / 0.25);
    b = b > 15 ? 15 : (b < 0 ? 0 : b);
    atomicAdd(&hist[j * 16 + b], 1u);
  }
}

__global__ void k_features_norm(const unsigned* __restrict__ hist, int n, int K, float* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = (float)((double)hist[i] / (double)K);
}

}  // namespace
}  // namespace gmco

using namespace gmco;

struct gmco_mlp {
  int device = 0;
  hipStream_t stream = nullptr;
  std::vector<int> sizes;
  int max_batch = 0;
  size_t n_params = 0;
  std::vector<size_t> woff, boff;  // parameter offsets per layer
  float *p = nullptr, *g = nullptr, *m = nullptr, *v = nullptr;
  std::vector<float*> act;   // act[0] = input, act[k+1] = output of layer k
  std::vector<float*> dact;  // gradient buffers, same shapes
  float* y = nullptr;        // targets of the batch
  double* loss = nullptr;
  float *dataX = nullptr, *dataY = nullptr;
  void* steps = nullptr;     // order, tile losses and losses of a training call
  size_t steps_bytes = 0;
  int n_data = 0;
  int adam_step = 0;
  std::vector<void*> owned;
  std::string err;
};

namespace {

int mfail(gmco_mlp* m, int code, const std::string& msg) {
  if (m) m->err = msg;
  return code;
}

#define MLP_HIP(mm, call)                                                             \
  do {                                                                                \
    hipError_t e_ = (call);                                                           \
    if (e_ != hipSuccess) return mfail((mm), GMCO_EHIP, std::string(#call) + ": " + hipGetErrorString(e_)); \
  } while (0)

int layers(const gmco_mlp* m) { return (int)m->sizes.size() - 1; }

int tiles_of(int rows, int cols, int T) { return ((rows + T - 1) / T) * ((cols + T - 1) / T); }

template <int FORM, bool WIDE>
hipError_t gemm_launch(hipStream_t st, const GemmArgs& a) {
  if constexpr (FORM != GEMM_FWD_MSE) {  // (whose tile losses are laid out for 32 x 32 tiles)
    if (tiles_of(a.M, a.N, 64) >= kGemmWide) {
      hipLaunchKernelGGL((k_gemm<64, FORM, WIDE>), dim3((a.M + 63) / 64, (a.N + 63) / 64), dim3(256), 0, st, a);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((k_gemm<32, FORM, WIDE>), dim3((a.M + 31) / 32, (a.N + 31) / 32), dim3(256), 0, st, a);
  return hipGetLastError();
}

// The operands that are contiguous in k (A, and B of the forward products) are
// read by whole float4 where their rows are of whole, aligned ones.
template <int FORM>
hipError_t gemm(hipStream_t st, const GemmArgs& a) {
  auto whole = [&](const float* p, int ld) { return ld % 4 == 0 && (reinterpret_cast<size_t>(p) & 15) == 0; };
  const bool wide = a.K % 4 == 0 && whole(a.A, a.lda) && (FORM > GEMM_FWD_MSE || whole(a.B, a.ldb));
  return wide ? gemm_launch<FORM, true>(st, a) : gemm_launch<FORM, false>(st, a);
}

GemmArgs forward_args(const gmco_mlp* m, int B, int k, const float* in, const int* rows) {
  GemmArgs a{};
  a.A = k == 0 ? in : m->act[k];
  a.rows = k == 0 ? rows : nullptr;
  a.gathered = m->act[0];
  a.B = m->p + m->woff[k];
  a.C = m->act[k + 1];
  a.bias = m->p + m->boff[k];
  a.lda = a.ldb = m->sizes[k];
  a.M = B;
  a.N = m->sizes[k + 1];
  a.K = m->sizes[k];
  a.relu = k < layers(m) - 1;
  return a;
}

// forward over B rows of `in` (row i at rows[i] if given): act[k+1] =
// relu?(act[k] W_k^T + b_k), on stream st (the network's own unless a
// caller's); layers 0 .. n - 1
hipError_t forward(gmco_mlp* m, int B, const float* in, const int* rows, int n, hipStream_t st) {
  for (int k = 0; k < n; ++k) {
    const hipError_t e = gemm<GEMM_FWD>(st, forward_args(m, B, k, in, rows));
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// One training step's products on B rows of `in` and `y` (at rows[i] if
// given): forward with the squared error's derivative and tile sums (into
// tile_loss), the activations' gradients, then every layer's weight and bias
// gradients into m->g, or, with ad, their Adam update of m->p.
hipError_t step_products(gmco_mlp* m, int B, const float* in, const float* y, const int* rows, double* tile_loss,
                         const AdamArgs* ad) {
  const int L = layers(m);
  hipError_t e = forward(m, B, in, rows, L - 1, m->stream);
  if (e != hipSuccess) return e;
  GemmArgs f = forward_args(m, B, L - 1, in, rows);
  f.C = m->dact[L];
  f.y = y;
  f.yrows = rows;
  f.loss = tile_loss;
  f.scale = 2.f / ((float)B * (float)m->sizes[L]);
  e = gemm<GEMM_FWD_MSE>(m->stream, f);
  if (e != hipSuccess) return e;
  for (int k = L - 1; k > 0; --k) {  // d act[k] = (G W_k) where act[k] > 0   (B x in)
    GemmArgs a{};
    a.A = m->dact[k + 1];
    a.B = m->p + m->woff[k];
    a.C = m->dact[k];
    a.act = m->act[k];
    a.lda = m->sizes[k + 1];
    a.ldb = m->sizes[k];
    a.M = B;
    a.N = m->sizes[k];
    a.K = m->sizes[k + 1];
    e = gemm<GEMM_DACT>(m->stream, a);
    if (e != hipSuccess) return e;
  }
  for (int k0 = 0; k0 < L; k0 += kDwLayers) {
    DwArgs d{};
    d.n = std::min(kDwLayers, L - k0);
    int wide = 0;
    for (int l = 0; l < d.n; ++l) wide += tiles_of(m->sizes[k0 + l + 1], m->sizes[k0 + l], 64);
    const int T = wide >= kGemmWide ? 64 : 32;
    for (int l = 0; l < d.n; ++l) {  // dW_k = G^T act[k]   (out x in), contraction over the batch
      const int k = k0 + l, out = m->sizes[k + 1], nin = m->sizes[k];
      GemmArgs& a = d.g[l];
      a.A = m->dact[k + 1];
      a.lda = out;
      a.B = k == 0 && !rows ? in : m->act[k];  // (gathered rows: written by the forward product)
      a.ldb = nin;
      a.M = out;
      a.N = nin;
      a.K = B;
      a.C = m->g + m->woff[k];
      a.p = m->p + m->woff[k];
      a.m = m->m + m->woff[k];
      a.v = m->v + m->woff[k];
      d.db[l] = (ad ? m->p : m->g) + m->boff[k];
      d.dbm[l] = m->m + m->boff[k];
      d.dbv[l] = m->v + m->boff[k];
      d.first[l + 1] = d.first[l] + tiles_of(out, nin, T) + (out + 63) / 64;
    }
    if (ad) d.ad = *ad;
    const dim3 grid(d.first[d.n]);
    if (ad && T == 64) hipLaunchKernelGGL((k_dw<64, true>), grid, dim3(256), 0, m->stream, d);
    else if (ad) hipLaunchKernelGGL((k_dw<32, true>), grid, dim3(256), 0, m->stream, d);
    else if (T == 64) hipLaunchKernelGGL((k_dw<64, false>), grid, dim3(256), 0, m->stream, d);
    else hipLaunchKernelGGL((k_dw<32, false>), grid, dim3(256), 0, m->stream, d);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

int loss_tiles(const gmco_mlp* m, int B) { return tiles_of(B, m->sizes.back(), 32); }

// Device memory of a training call, kept for the next one and grown when a
// call needs more (its last work has ended: every call synchronises).  The order
// of a long call is as long as the call, so past kStepsKeep it goes back when the
// call returns.
constexpr size_t kStepsKeep = size_t(16) << 20;

void release_steps(gmco_mlp* m) {
  if (!m->steps) return;
  m->owned.erase(std::find(m->owned.begin(), m->owned.end(), m->steps));
  (void)hipFree(m->steps);
  m->steps = nullptr;
  m->steps_bytes = 0;
}

hipError_t reserve_steps(gmco_mlp* m, size_t bytes) {
  if (m->steps_bytes >= bytes) return hipSuccess;
  release_steps(m);
  void* p = nullptr;
  const hipError_t e = hipMalloc(&p, bytes);
  if (e != hipSuccess) return e;
  m->owned.push_back(p);
  m->steps = p;
  m->steps_bytes = bytes;
  return hipSuccess;
}

}  // namespace

extern "C" {

int gmco_mlp_create(gmco_mlp** out, int device, const int* sizes, int n_sizes, int max_batch) {
  if (!out || !sizes || n_sizes < 2 || max_batch < 1) return GMCO_EINVAL;
  *out = nullptr;
  for (int k = 0; k < n_sizes; ++k)
    if (sizes[k] < 1 || sizes[k] > 4096) return GMCO_EINVAL;
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || ndev <= 0) return GMCO_ENOLIB;
  if (device < 0 || device >= ndev) return GMCO_EINVAL;
  if (hipSetDevice(device) != hipSuccess) return GMCO_EHIP;
  gmco_mlp* m = new (std::nothrow) gmco_mlp();
  if (!m) return GMCO_ENOMEM;
  m->device = device;
  m->sizes.assign(sizes, sizes + n_sizes);
  m->max_batch = max_batch;
  size_t off = 0;
  for (int k = 0; k + 1 < n_sizes; ++k) {
    m->woff.push_back(off);
    off += (size_t)sizes[k] * sizes[k + 1];
    m->boff.push_back(off);
    off += (size_t)sizes[k + 1];
  }
  m->n_params = off;
  auto alloc = [&](size_t bytes) -> void* {
    void* ptr = nullptr;
    if (hipMalloc(&ptr, std::max<size_t>(bytes, 256)) != hipSuccess) return nullptr;
    m->owned.push_back(ptr);
    return ptr;
  };
  bool ok = true;
  m->p = (float*)alloc(off * 4);
  m->g = (float*)alloc(off * 4);
  m->m = (float*)alloc(off * 4);
  m->v = (float*)alloc(off * 4);
  for (int k = 0; k < n_sizes; ++k) {
    m->act.push_back((float*)alloc((size_t)max_batch * sizes[k] * 4));
    m->dact.push_back((float*)alloc((size_t)max_batch * sizes[k] * 4));
  }
  m->y = (float*)alloc((size_t)max_batch * sizes[n_sizes - 1] * 4);
  m->loss = (double*)alloc((size_t)(1 + loss_tiles(m, max_batch)) * 8);  // the loss, then its tiles
  for (void* ptr : m->owned) ok = ok && ptr;
  if (!ok || hipMemset(m->p, 0, off * 4) != hipSuccess || hipMemset(m->m, 0, off * 4) != hipSuccess ||
      hipMemset(m->v, 0, off * 4) != hipSuccess) {
    gmco_mlp_destroy(m);
    return GMCO_ENOMEM;
  }
  *out = m;
  return GMCO_OK;
}

int gmco_mlp_destroy(gmco_mlp* m) {
  if (!m) return GMCO_OK;
  hipSetDevice(m->device);
  hipDeviceSynchronize();
  for (void* ptr : m->owned) hipFree(ptr);
  delete m;
  return GMCO_OK;
}

int gmco_mlp_set_stream(gmco_mlp* m, void* stream) {
  if (!m) return GMCO_EINVAL;
  m->stream = (hipStream_t)stream;
  return GMCO_OK;
}

int gmco_mlp_param_count(const gmco_mlp* m, size_t* n) {
  if (!m || !n) return GMCO_EINVAL;
  *n = m->n_params;
  return GMCO_OK;
}

const char* gmco_mlp_last_error(const gmco_mlp* m) { return m ? m->err.c_str() : "null network"; }

int gmco_mlp_set_params(gmco_mlp* m, const float* p, size_t n) {
  if (!m || !p || n != m->n_params) return GMCO_EINVAL;
  MLP_HIP(m, hipSetDevice(m->device));
  MLP_HIP(m, hipMemcpyAsync(m->p, p, n * 4, hipMemcpyHostToDevice, m->stream));
  MLP_HIP(m, hipMemsetAsync(m->m, 0, n * 4, m->stream));
  MLP_HIP(m, hipMemsetAsync(m->v, 0, n * 4, m->stream));
  MLP_HIP(m, hipStreamSynchronize(m->stream));
  m->adam_step = 0;
  return GMCO_OK;
}

int gmco_mlp_get_params(gmco_mlp* m, float* p, size_t n) {
  if (!m || !p || n != m->n_params) return GMCO_EINVAL;
  MLP_HIP(m, hipSetDevice(m->device));
  MLP_HIP(m, hipMemcpyAsync(p, m->p, n * 4, hipMemcpyDeviceToHost, m->stream));
  MLP_HIP(m, hipStreamSynchronize(m->stream));
  return GMCO_OK;
}

int gmco_mlp_loss_grad(gmco_mlp* m, int B, const float* X, const float* Y, double* loss, float* grad) {
  if (!m || !X || !Y || B < 1 || B > m->max_batch) return GMCO_EINVAL;
  MLP_HIP(m, hipSetDevice(m->device));
  const int L = layers(m);
  MLP_HIP(m, hipMemcpyAsync(m->act[0], X, (size_t)B * m->sizes[0] * 4, hipMemcpyHostToDevice, m->stream));
  MLP_HIP(m, hipMemcpyAsync(m->y, Y, (size_t)B * m->sizes[L] * 4, hipMemcpyHostToDevice, m->stream));
  MLP_HIP(m, step_products(m, B, m->act[0], m->y, nullptr, m->loss + 1, nullptr));
  hipLaunchKernelGGL(k_sum_loss, dim3(1), dim3(256), 0, m->stream, m->loss + 1, loss_tiles(m, B),
                     (double)B * (double)m->sizes[L], m->loss);
  MLP_HIP(m, hipGetLastError());
  if (loss) MLP_HIP(m, hipMemcpyAsync(loss, m->loss, 8, hipMemcpyDeviceToHost, m->stream));
  if (grad) MLP_HIP(m, hipMemcpyAsync(grad, m->g, m->n_params * 4, hipMemcpyDeviceToHost, m->stream));
  MLP_HIP(m, hipStreamSynchronize(m->stream));
  return GMCO_OK;
}

int gmco_mlp_set_data(gmco_mlp* m, int N, const float* X, const float* Y) {
  if (!m || N < 1 || !X || !Y) return GMCO_EINVAL;
  MLP_HIP(m, hipSetDevice(m->device));
  const int L = layers(m);
  for (float* ptr : {m->dataX, m->dataY}) {
    if (ptr) {
      m->owned.erase(std::find(m->owned.begin(), m->owned.end(), (void*)ptr));
      hipFree(ptr);
    }
  }
  m->dataX = m->dataY = nullptr;
  m->n_data = 0;
  void *dx = nullptr, *dy = nullptr;
  if (hipMalloc(&dx, (size_t)N * m->sizes[0] * 4) != hipSuccess) return mfail(m, GMCO_ENOMEM, "data X");
  m->owned.push_back(dx);
  if (hipMalloc(&dy, (size_t)N * m->sizes[L] * 4) != hipSuccess) return mfail(m, GMCO_ENOMEM, "data Y");
  m->owned.push_back(dy);
  m->dataX = (float*)dx;
  m->dataY = (float*)dy;
  MLP_HIP(m, hipMemcpyAsync(dx, X, (size_t)N * m->sizes[0] * 4, hipMemcpyHostToDevice, m->stream));
  MLP_HIP(m, hipMemcpyAsync(dy, Y, (size_t)N * m->sizes[L] * 4, hipMemcpyHostToDevice, m->stream));
  MLP_HIP(m, hipStreamSynchronize(m->stream));
  m->n_data = N;
  return GMCO_OK;
}

int gmco_mlp_train(gmco_mlp* m, int n_steps, int B, const int32_t* order, float lr, double* mean_loss) {
  if (!m || !order || n_steps < 1 || B < 1 || B > m->max_batch || !(lr > 0.f)) return GMCO_EINVAL;
  if (m->n_data == 0) return mfail(m, GMCO_ESTATE, "gmco_mlp_set_data first");
  for (size_t i = 0; i < (size_t)n_steps * B; ++i)
    if (order[i] < 0 || order[i] >= m->n_data) return mfail(m, GMCO_EINVAL, "sample index out of range");
  MLP_HIP(m, hipSetDevice(m->device));
  const int L = layers(m);
  const int nt = loss_tiles(m, B);
  const size_t order_bytes = ((size_t)n_steps * B * 4 + 255) / 256 * 256;
  // tile losses of up to kLossSteps steps, reduced together
  constexpr int kLossSteps = 64;
  if (reserve_steps(m, order_bytes + ((size_t)n_steps + (size_t)std::min(n_steps, kLossSteps) * nt) * 8) != hipSuccess)
    return mfail(m, GMCO_ENOMEM, "training buffers");
  struct Release {
    gmco_mlp* m;
    ~Release() {
      if (m->steps_bytes > kStepsKeep) release_steps(m);
    }
  } release{m};
  int* dorder = (int*)m->steps;
  double* losses = (double*)((char*)m->steps + order_bytes);
  double* tile_loss = losses + n_steps;
  MLP_HIP(m, hipMemcpyAsync(dorder, order, (size_t)n_steps * B * 4, hipMemcpyHostToDevice, m->stream));
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  for (int s = 0; s < n_steps; ++s) {
    m->adam_step += 1;
    const AdamArgs ad{lr, b1, b2, eps, 1.f - powf(b1, (float)m->adam_step), 1.f - powf(b2, (float)m->adam_step)};
    MLP_HIP(m, step_products(m, B, m->dataX, m->dataY, dorder + (size_t)s * B,
                             tile_loss + (size_t)(s % kLossSteps) * nt, &ad));
    if (s + 1 == n_steps || (s + 1) % kLossSteps == 0) {
      const int first = s / kLossSteps * kLossSteps;
      hipLaunchKernelGGL(k_sum_loss, dim3(s + 1 - first), dim3(256), 0, m->stream, tile_loss, nt,
                         (double)B * (double)m->sizes[L], losses + first);
      MLP_HIP(m, hipGetLastError());
    }
  }
  std::vector<double> h(n_steps);
  MLP_HIP(m, hipMemcpyAsync(h.data(), losses, (size_t)n_steps * 8, hipMemcpyDeviceToHost, m->stream));
  MLP_HIP(m, hipStreamSynchronize(m->stream));
  if (mean_loss) {
    double s = 0.0;
    for (double v : h) s += v;
    *mean_loss = s / n_steps;
  }
  return GMCO_OK;
}

int gmco_mlp_predict(gmco_mlp* m, int B, const float* X, float* Y) {
  if (!m || !X || !Y || B < 1) return GMCO_EINVAL;
  MLP_HIP(m, hipSetDevice(m->device));
  const int L = layers(m);
  for (int b0 = 0; b0 < B; b0 += m->max_batch) {
    const int nb = std::min(m->max_batch, B - b0);
    MLP_HIP(m, hipMemcpyAsync(m->act[0], X + (size_t)b0 * m->sizes[0], (size_t)nb * m->sizes[0] * 4,
                              hipMemcpyHostToDevice, m->stream));
    MLP_HIP(m, forward(m, nb, m->act[0], nullptr, L, m->stream));
    MLP_HIP(m, hipMemcpyAsync(Y + (size_t)b0 * m->sizes[L], m->act[L], (size_t)nb * m->sizes[L] * 4,
                              hipMemcpyDeviceToHost, m->stream));
  }
  MLP_HIP(m, hipStreamSynchronize(m->stream));
  return GMCO_OK;
}

}  // extern "C"

namespace gmco {
int mlp_inputs(const gmco_mlp* m) { return m->sizes.front(); }
int mlp_outputs(const gmco_mlp* m) { return m->sizes.back(); }
int mlp_device(const gmco_mlp* m) { return m->device; }

// The network on B rows held in device memory (X: B x n_in, Y: B x n_out),
// in chunks of max_batch rows, all on stream st.  The network's activation
// buffers are used, so st must be ordered with the network's other work.
hipError_t mlp_forward_device(gmco_mlp* m, int B, const float* X, float* Y, hipStream_t st) {
  const int L = layers(m);
  for (int b0 = 0; b0 < B; b0 += m->max_batch) {
    const int nb = std::min(m->max_batch, B - b0);
    hipError_t e = forward(m, nb, X + (size_t)b0 * m->sizes[0], nullptr, L, st);
    if (e != hipSuccess) return e;
    e = hipMemcpyAsync(Y + (size_t)b0 * m->sizes[L], m->act[L], (size_t)nb * m->sizes[L] * 4,
                       hipMemcpyDeviceToDevice, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_features(const double* dwell, const double* pts, const int* perm, const int* goff,
                           const int* gcnt, int K, int G, unsigned* hist, float* out, hipStream_t st) {
  hipError_t e = hipMemsetAsync(hist, 0, (size_t)G * 16 * 4, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_features, dim3(K, G), dim3(256), 0, st, dwell, pts, perm, goff, gcnt, K, hist);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_features_norm, dim3(1), dim3(256), 0, st, hist, G * 16, K, out);
  return hipGetLastError();
}
}  // namespace gmco
