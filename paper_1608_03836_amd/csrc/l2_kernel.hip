// Per-slice L2 norms with the element maps' Jacobians (the norm of the L2
// errors of Section 5.2), on the tiled state layout:
//
//   ||A_s - B_s||^2 = sum_k sum_q w_q J_kq sum_f ((V_q (A_s - B_s)_f)_kq)^2
//
// over the context's volume rule (q = i + nq j, w_q = w_i w_j), and ||B_s||^2
// likewise.  One workgroup per (slice, 64-element group) item, one element per
// lane: the field values are interpolated to the quadrature points by the
// tensor-product operator V (rows in r, then in s), squared and weighted by
// w_q J_q = w_q / (1/J)_q from the geometry.  Padding lanes contribute
// nothing.  Each item's two sums go to `partials` [S * nEG][2]; a second
// kernel adds a slice's partials in a fixed order (no atomics), so the result
// is bitwise reproducible.
//
// Bound by HBM, given enough loads in flight.  In general there is one wave
// per field, which share the divisions through LDS while their values arrive
// -- and at N >= 3 one for each of A - B and B, which reads B twice but halves
// the registers: 64x64 elements, N = 3, 64 slices of A and B (201 MB) took 63
// us with one wave per item, 44 with one per field, 39.6 with one per field
// and array (5.1 TB/s).  At N <= 2 that is slower than one per field (a call on
// 128x128 elements, N = 2, nq1 = 3, 200 slices: 298 us, 253; one wave per item
// 262), and at N = 1, nq1 <= 3, four values a field and few divisions, both
// are slower than one wave per item (nq1 = 3: 205, 158, 141; nq1 = 4: 230,
// 192, 185, but of 4 slices 38, 37, 37 and of A alone 132, 134, 146).

#include <hip/hip_runtime.h>

#include "reference_tables.h"
#include "stage_common.h"
#include "wadg_internal.h"

namespace wadg {
namespace {

using namespace dev;

// sum_q wj_q ((V (x) V) x)_q^2 for one field's nodal values x of this lane,
// wj_q = wj[q STRIDE].
template <int N, int NQ, int STRIDE>
__device__ __forceinline__ double quad_square(const double (&x)[(N + 1) * (N + 1)],
                                              const double* wj) {
  constexpr ct::Ops<double, N, NQ> T = ct::make_ops<double, N, NQ>();
  constexpr int NP1 = N + 1;
  double t[NP1][NQ];
#pragma unroll
  for (int b = 0; b < NP1; ++b)
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      double s = 0.0;
#pragma unroll
      for (int a = 0; a < NP1; ++a) s = mad(T.V[i][a], x[a + NP1 * b], s);
      t[b][i] = s;
    }
  double acc = 0.0;
#pragma unroll
  for (int j = 0; j < NQ; ++j)
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      double v = 0.0;
#pragma unroll
      for (int b = 0; b < NP1; ++b) v = mad(T.V[j][b], t[b][i], v);
      acc = mad(wj[(i + NQ * j) * STRIDE], v * v, acc);
    }
  return acc;
}

// Workgroup b of either kernel: item item0 + b.  PAIRED: B is there, else its
// sums are zero.

// One wave per item (N = 1, nq1 <= 3).
template <int N, int NQ, bool PAIRED>
__global__ __launch_bounds__(kWave) void l2_item_kernel(
    const double* __restrict__ A, const double* __restrict__ B, const double* __restrict__ vol,
    int item0, int nEG, int K, double* __restrict__ partials) {
  constexpr ct::Tables<N, NQ> tb = ct::make_tables<N, NQ>();
  constexpr int NP = (N + 1) * (N + 1), NQ2 = NQ * NQ;
  constexpr size_t tile = (size_t)3 * NP * kWave;
  const int item = item0 + (int)blockIdx.x;
  const int s = item / nEG, g = item - s * nEG;
  const int lane = threadIdx.x;
  const bool active = g * kWave + lane < K;
  const size_t off = ((size_t)s * nEG + g) * tile + lane;
  const double* a = A + off;
  const double* b = B + off;
  const double* inv_j = vol + ((size_t)g * 6 * NQ2 + 5 * NQ2) * kWave + lane;
  double wj[NQ2];
#pragma unroll
  for (int q = 0; q < NQ2; ++q)
    wj[q] = active ? (tb.wq[q % NQ] * tb.wq[q / NQ]) / inv_j[q * kWave] : 0.0;
  double sd = 0.0, sb = 0.0;
#pragma unroll
  for (int f = 0; f < 3; ++f) {
    double d[NP], e[NP];
#pragma unroll
    for (int n = 0; n < NP; ++n) {
      e[n] = PAIRED ? b[(f * NP + n) * kWave] : 0.0;
      d[n] = a[(f * NP + n) * kWave] - e[n];
    }
    sd += quad_square<N, NQ, 1>(d, wj);
    if (PAIRED) sb += quad_square<N, NQ, 1>(e, wj);
  }
  // padding lanes may hold anything (their weights are zero, but 0 * inf
  // is not): they are dropped here
  if (!active) sd = sb = 0.0;
#pragma unroll
  for (int o = kWave / 2; o >= 1; o >>= 1) {
    sd += __shfl_xor(sd, o, kWave);
    sb += __shfl_xor(sb, o, kWave);
  }
  if (lane == 0) {
    partials[2 * (size_t)item] = sd;
    partials[2 * (size_t)item + 1] = sb;
  }
}

// A wave per field f of an item, which forms A - B and B, or (N >= 3, B there)
// wave f of A - B and wave 3 + f of B.
template <int N, bool PAIRED>
struct FieldWaves {
  static constexpr bool both = PAIRED && N <= 2;
  static constexpr int n = PAIRED && !both ? 6 : 3;
};

template <int N, int NQ, bool PAIRED>
__global__ __launch_bounds__((FieldWaves<N, PAIRED>::n * kWave)) void l2_field_kernel(
    const double* __restrict__ A, const double* __restrict__ B, const double* __restrict__ vol,
    int item0, int nEG, int K, double* __restrict__ partials) {
  constexpr ct::Tables<N, NQ> tb = ct::make_tables<N, NQ>();
  constexpr int NP = (N + 1) * (N + 1), NQ2 = NQ * NQ, W = FieldWaves<N, PAIRED>::n;
  constexpr bool both = FieldWaves<N, PAIRED>::both;
  constexpr size_t tile = (size_t)3 * NP * kWave;
  __shared__ double wj[NQ2 * kWave];
  __shared__ double part[6];
  const int item = item0 + (int)blockIdx.x;
  const int s = item / nEG, g = item - s * nEG;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int f = w % 3;
  const bool active = g * kWave + lane < K;
  const size_t off = ((size_t)s * nEG + g) * tile + (size_t)f * NP * kWave + lane;
  const double* a = (w < 3 ? A : B) + off;
  double x[NP], y[both ? NP : 1];
#pragma unroll
  for (int n = 0; n < NP; ++n) x[n] = a[n * kWave];
  if (PAIRED && w < 3) {
    const double* b = B + off;
#pragma unroll
    for (int n = 0; n < NP; ++n) {
      const double bv = b[n * kWave];
      x[n] -= bv;
      if constexpr (both) y[n] = bv;
    }
  }
  const double* inv_j = vol + ((size_t)g * 6 * NQ2 + 5 * NQ2) * kWave + lane;
#pragma unroll
  for (int q0 = 0; q0 < NQ2; q0 += W) {
    const int q = q0 + w;
    if (q < NQ2)
      wj[q * kWave + lane] =
          active ? (tb.wq[q % NQ] * tb.wq[q / NQ]) / inv_j[q * kWave] : 0.0;
  }
  if (threadIdx.x < 6) part[threadIdx.x] = 0.0;
  __syncthreads();
  // (padding lanes dropped as above)
  auto item_sum = [&](const auto& v) {
    double sum = quad_square<N, NQ, kWave>(v, wj + lane);
    if (!active) sum = 0.0;
#pragma unroll
    for (int o = kWave / 2; o >= 1; o >>= 1) sum += __shfl_xor(sum, o, kWave);
    return sum;
  };
  const double sum = item_sum(x);
  if (lane == 0) part[w] = sum;
  if constexpr (both) {
    const double sb = item_sum(y);
    if (lane == 0) part[3 + w] = sb;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    const double* r = part + 3 * threadIdx.x;
    partials[2 * (size_t)item + threadIdx.x] = r[0] + r[1] + r[2];
  }
}

// One wave per slice: each lane adds a strided run of the slice's item
// partials in order, four of them in flight, then the wave's tree.
__global__ __launch_bounds__(kWave) void l2_final_kernel(const double* __restrict__ partials,
                                                         int nEG, double* __restrict__ out) {
  const int s = blockIdx.x, lane = threadIdx.x;
  const double* p = partials + 2 * (size_t)s * nEG;
  double sd = 0.0, sb = 0.0;
  constexpr int U = 4;
  for (int64_t g0 = lane; g0 < nEG; g0 += U * kWave) {
    double d[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t g = g0 + u * kWave, at = g < nEG ? g : g0;
      d[u] = p[2 * at];
      b[u] = p[2 * at + 1];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (g0 + u * kWave < nEG) {
        sd += d[u];
        sb += b[u];
      }
  }
#pragma unroll
  for (int o = kWave / 2; o >= 1; o >>= 1) {
    sd += __shfl_xor(sd, o, kWave);
    sb += __shfl_xor(sb, o, kWave);
  }
  if (lane == 0) {
    out[2 * (size_t)s] = sd;
    out[2 * (size_t)s + 1] = sb;
  }
}

template <int N, int NQ, bool PAIRED>
int launch_items(const double* A, const double* B, const double* vol, int32_t S, int32_t nEG,
                 int32_t K, double* partials, hipStream_t st) {
  constexpr bool whole = N == 1 && NQ <= 3;
  constexpr int threads = (whole ? 1 : FieldWaves<N, PAIRED>::n) * kWave;
  // (HIP takes fewer than 2^32 lanes per launch: 11 million items at six waves)
  const int64_t most = ((1LL << 32) - 1) / threads, items = (int64_t)S * nEG;
  for (int64_t i = 0; i < items; i += most) {
    const dim3 grid((unsigned)(items - i < most ? items - i : most));
    if constexpr (whole)
      hipLaunchKernelGGL((l2_item_kernel<N, NQ, PAIRED>), grid, dim3(threads), 0, st, A, B, vol,
                         (int)i, nEG, K, partials);
    else
      hipLaunchKernelGGL((l2_field_kernel<N, NQ, PAIRED>), grid, dim3(threads), 0, st, A, B, vol,
                         (int)i, nEG, K, partials);
    const int e = (int)hipGetLastError();
    if (e) return e;
  }
  return 0;
}

template <int N, int NQ>
int launch_nq(const double* A, const double* B, const double* vol, int32_t S, int32_t nEG,
              int32_t K, double* partials, double* out, hipStream_t st) {
  const int e = B ? launch_items<N, NQ, true>(A, B, vol, S, nEG, K, partials, st)
                  : launch_items<N, NQ, false>(A, A, vol, S, nEG, K, partials, st);
  if (e) return e;
  hipLaunchKernelGGL(l2_final_kernel, dim3(S), dim3(kWave), 0, st, partials, nEG, out);
  return (int)hipGetLastError();
}

template <int N>
int launch_n(int nq, const double* A, const double* B, const double* vol, int32_t S,
             int32_t nEG, int32_t K, double* partials, double* out, hipStream_t st) {
  switch (nq - N) {
    case 1: return launch_nq<N, N + 1>(A, B, vol, S, nEG, K, partials, out, st);
    case 2: return launch_nq<N, N + 2>(A, B, vol, S, nEG, K, partials, out, st);
    case 3: return launch_nq<N, N + 3>(A, B, vol, S, nEG, K, partials, out, st);
    default: return (int)hipErrorInvalidValue;
  }
}

}  // namespace

int launch_l2_norms(int N, int nq, const double* A, const double* B, const double* vol,
                    int32_t S, int32_t nEG, int32_t K, double* partials, double* out,
                    void* stream) {
  if (S < 1 || nEG < 1 || (int64_t)S * nEG > INT32_MAX) return (int)hipErrorInvalidValue;
  hipStream_t st = static_cast<hipStream_t>(stream);
  switch (N) {
    case 1: return launch_n<1>(nq, A, B, vol, S, nEG, K, partials, out, st);
    case 2: return launch_n<2>(nq, A, B, vol, S, nEG, K, partials, out, st);
    case 3: return launch_n<3>(nq, A, B, vol, S, nEG, K, partials, out, st);
    case 4: return launch_n<4>(nq, A, B, vol, S, nEG, K, partials, out, st);
    default: return (int)hipErrorInvalidValue;
  }
}

}  // namespace wadg
