// Per-slice L2 norms with the element maps' Jacobians (the norm of the L2
// errors of Section 5.2), on the tiled state layout:
//
//   ||A_s - B_s||^2 = sum_k sum_q w_q J_kq sum_f ((V_q (A_s - B_s)_f)_kq)^2
//
// over the context's volume rule (q = i + nq j, w_q = w_i w_j), and ||B_s||^2
// likewise.  One workgroup per (slice, 64-element group) item, one element
// per lane and one wave per field of A - B and of B: the field values are
// interpolated to the quadrature points by the tensor-product operator V
// (rows in r, then in s), squared and weighted by w_q J_q = w_q / (1/J)_q
// from the geometry, whose divisions the waves share through LDS while their
// values arrive.  Padding lanes contribute nothing.  Each item's two sums go
// to `partials` [S * nEG][2]; a second kernel adds a slice's partials in a
// fixed order (no atomics), so the result is bitwise reproducible.
//
// Bound by HBM, given enough loads in flight: with one wave per item (all
// fields one after another, and every division) 64x64 elements, N = 3, 64
// slices of A and B (201 MB) took 63 us; one wave per field 44 us; one per
// field and array, which reads B twice but half the registers, 39.6 us (5.1
// TB/s).

#include <hip/hip_runtime.h>

#include "reference_tables.h"
#include "stage_common.h"
#include "wadg_internal.h"

namespace wadg {
namespace {

using namespace dev;

// sum_q wj_q ((V (x) V) x)_q^2 for one field's nodal values x of this lane,
// wj_q = wj[q * 64].
template <int N, int NQ>
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
      acc = mad(wj[(i + NQ * j) * kWave], v * v, acc);
    }
  return acc;
}

// PAIRED: six waves, field f's A - B by wave f and its B by wave 3 + f;
// else B is absent, and three waves.  Workgroup b: item item0 + b.
template <int N, int NQ, bool PAIRED>
__global__ __launch_bounds__((PAIRED ? 6 : 3) * kWave) void l2_partial_kernel(
    const double* __restrict__ A, const double* __restrict__ B, const double* __restrict__ vol,
    int item0, int nEG, int K, double* __restrict__ partials) {
  constexpr ct::Tables<N, NQ> tb = ct::make_tables<N, NQ>();
  constexpr int NP = (N + 1) * (N + 1), NQ2 = NQ * NQ, W = PAIRED ? 6 : 3;
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
  double x[NP];
#pragma unroll
  for (int n = 0; n < NP; ++n) x[n] = a[n * kWave];
  if (PAIRED && w < 3) {
    const double* b = B + off;
#pragma unroll
    for (int n = 0; n < NP; ++n) x[n] -= b[n * kWave];
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
  // padding lanes may hold anything (their weights are zero, but 0 * inf
  // is not): they are dropped here
  double sum = quad_square<N, NQ>(x, wj + lane);
  if (!active) sum = 0.0;
#pragma unroll
  for (int o = kWave / 2; o >= 1; o >>= 1) sum += __shfl_xor(sum, o, kWave);
  if (lane == 0) part[w] = sum;
  __syncthreads();
  if (threadIdx.x < 2) {
    const double* r = part + 3 * threadIdx.x;
    partials[2 * (size_t)item + threadIdx.x] = r[0] + r[1] + r[2];
  }
}

// One wave per slice: each lane adds a strided run of the slice's item
// partials in order, then the wave's tree.
__global__ __launch_bounds__(kWave) void l2_final_kernel(const double* __restrict__ partials,
                                                         int nEG, double* __restrict__ out) {
  const int s = blockIdx.x, lane = threadIdx.x;
  const double* p = partials + 2 * (size_t)s * nEG;
  double sd = 0.0, sb = 0.0;
  for (int g = lane; g < nEG; g += kWave) {
    sd += p[2 * (size_t)g];
    sb += p[2 * (size_t)g + 1];
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

template <int N, int NQ>
int launch_nq(const double* A, const double* B, const double* vol, int32_t S, int32_t nEG,
              int32_t K, double* partials, double* out, hipStream_t st) {
  // (HIP takes fewer than 2^32 lanes per launch: 11 million items at six waves)
  const int threads = (B ? 6 : 3) * kWave;
  const int64_t most = ((1LL << 32) - 1) / threads, items = (int64_t)S * nEG;
  for (int64_t i = 0; i < items; i += most) {
    const dim3 grid((unsigned)(items - i < most ? items - i : most));
    if (B)
      hipLaunchKernelGGL((l2_partial_kernel<N, NQ, true>), grid, dim3(threads), 0, st, A, B, vol,
                         (int)i, nEG, K, partials);
    else
      hipLaunchKernelGGL((l2_partial_kernel<N, NQ, false>), grid, dim3(threads), 0, st, A, A, vol,
                         (int)i, nEG, K, partials);
    const int e = (int)hipGetLastError();
    if (e) return e;
  }
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
