// Stochastic Lanczos quadrature of ln|A| from the CG coefficients (the
// stochastic log-determinant discussed in Sec. 3.3 for eq. "gp-mll").
//
// For probe j the k x k tridiagonal T implied by CG, T_kk = 1/a_k + b_{k-1}/a_{k-1},
// T_{k,k+1} = sqrt(b_k)/a_k, gives z^T ln(A) z ~= |z|^2 e_1^T ln(T) e_1 (Gauss
// quadrature on the Ritz values). Instead of diagonalising T, the quadratic form
// is evaluated from the integral representation of the logarithm,
//   ln x = int_R e^s [ 1/(1 + e^s) - 1/(x + e^s) ] ds,
// so e_1^T ln(T) e_1 = int e^s [ 1/(1 + e^s) - e_1^T (T + e^s I)^{-1} e_1 ] ds.
// The integrand is analytic in the strip |Im s| < pi (poles at s = ln x + i pi),
// so the trapezoidal rule with step h converges like exp(-2 pi^2 / h); nodes run
// from ln(x_hi) - 75 to ln(x_hi) + 38 (x_hi a Gershgorin bound), where the
// integrand is below 1e-16. Each resolvent element (T + tI)^{-1}_{11} is a
// continued fraction evaluated from the bottom of T (the pivots of an LDL^T
// factorisation, all positive for t >= 0 when T is positive definite).
// One workgroup per probe: the coefficients sit in LDS, a thread takes a node (a chain of
// as many FP64 divisions as T has rows, which is what bounds the kernel), one more the
// test that T is positive definite, and a fixed-order reduction sums the nodes (FP64
// throughout). One wave per probe, five nodes a lane after the test and the bound by
// lane 0, took 415 us for some 700 rows; 69 us now.
#include <cmath>

#include "common.hpp"

namespace gpl {

constexpr int kSlqMaxSteps = 4096;       // LDS capacity per probe (doubles x 2)
constexpr double kSlqStep = 0.4;         // trapezoid step in s = ln t
constexpr double kSlqLo = 75.0, kSlqHi = 38.0;

constexpr int kSlqNodes = (int)((kSlqLo + kSlqHi) / kSlqStep) + 1;
constexpr int kSlqThreads = (kSlqNodes + 1 + 63) / 64 * 64;

__global__ __launch_bounds__(kSlqThreads) void slq_probe_kernel(int nprobe, int n_lanczos,
                                                                const double* __restrict__ ab,
                                                                const int* __restrict__ iters,
                                                                const double* __restrict__ bnorm2, double* contrib) {
  __shared__ double diag[kSlqMaxSteps];
  __shared__ double off2[kSlqMaxSteps];
  __shared__ double node_t[kSlqThreads], node_f[kSlqThreads];
  __shared__ double red[kSlqThreads / 64];
  __shared__ int s_ok;
  const int j = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int m = min(iters[j], n_lanczos);
  if (m <= 0) {
    if (tid == 0) contrib[j] = 0.0;
    return;
  }
  const double* a = ab + (size_t)j * n_lanczos * 2;
  for (int k = tid; k < m; k += kSlqThreads) {
    const double ak = a[2 * k], bk = a[2 * k + 1];
    double dk = 1.0 / ak;
    if (k > 0) dk += a[2 * (k - 1) + 1] / a[2 * (k - 1)];
    diag[k] = dk;
    off2[k] = (k + 1 < m) ? bk / (ak * ak) : 0.0;  // (sqrt(b_k)/a_k)^2
  }
  __syncthreads();
  // Gershgorin upper bound of the spectrum (fmax passes over a NaN)
  double hi = -INFINITY;
  for (int k = tid; k < m; k += kSlqThreads)
    hi = fmax(hi, diag[k] + ((k + 1 < m ? sqrt(off2[k]) : 0.0) + (k > 0 ? sqrt(off2[k - 1]) : 0.0)));
  for (int off = 32; off > 0; off >>= 1) hi = fmax(hi, __shfl_xor(hi, off, 64));
  if (lane == 0) red[tid >> 6] = hi;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kSlqThreads / 64; ++w) hi = fmax(hi, red[w]);
  const double s_lo = log(hi) - kSlqLo;
  {
    // (T + t I)^{-1}_{11} by the pivots from the bottom of T; the thread after the
    // nodes, with t = 0, looks whether all of them are positive
    const bool test = tid == kSlqNodes;
    const double t = test ? 0.0 : exp(s_lo + tid * kSlqStep);
    double g = diag[m - 1] + t;
    int ok = g > 0.0;
    for (int k = m - 2; k >= 0; --k) {
      g = (diag[k] + t) - off2[k] / g;
      ok &= g > 0.0;
    }
    if (test) s_ok = ok && isfinite(g);
    node_t[tid] = t;
    node_f[tid] = 1.0 / (1.0 + t) - 1.0 / g;
  }
  __syncthreads();
  if (tid >= 64) return;
  if (!s_ok) {
    if (lane == 0) contrib[j] = __builtin_nan("");
    return;
  }
  double acc = 0.0;
  for (int q = lane; q < kSlqNodes; q += 64) acc += node_t[q] * node_f[q];
  acc = warp_sum(acc);
  if (lane == 0) contrib[j] = bnorm2[j] * kSlqStep * acc;
}

__global__ void slq_sum_kernel(int nprobe, double scale, const double* offset, const double* contrib, double* logdet,
                               double* stderr_out) {
  if (threadIdx.x != 0) return;
  double s = 0.0;
  for (int j = 0; j < nprobe; ++j) s += contrib[j];
  const double mean = s / nprobe;
  double v = 0.0;
  for (int j = 0; j < nprobe; ++j) v += (contrib[j] - mean) * (contrib[j] - mean);
  *logdet = scale * s + (offset ? *offset : 0.0);
  // sample standard deviation of the contributions, scaled like the estimate
  *stderr_out = nprobe > 1 ? scale * sqrt(v / (nprobe - 1)) * sqrt((double)nprobe) : NAN;
}

}  // namespace gpl

using namespace gpl;

extern "C" size_t gpl_lanczos_logdet_workspace(int nprobe, int n_lanczos) {
  (void)nprobe;
  (void)n_lanczos;
  return 0;  // coefficients are staged in LDS
}

extern "C" int gpl_lanczos_logdet(int nprobe, int n_lanczos, const double* lanczos_ab, const int* iters,
                                  const double* bnorm2, double scale, const double* offset, double* contrib,
                                  double* logdet, double* stderr_out, void* ws, size_t ws_bytes,
                                  hipStream_t stream) {
  GPL_REQUIRE(nprobe >= 1 && n_lanczos >= 1, "nprobe=%d n_lanczos=%d must be >= 1", nprobe, n_lanczos);
  GPL_REQUIRE(lanczos_ab && iters && bnorm2 && contrib && logdet && stderr_out, "NULL argument");
  GPL_REQUIRE(std::isfinite(scale), "scale must be finite");
  GPL_REQUIRE(n_lanczos <= kSlqMaxSteps, "n_lanczos=%d exceeds %d", n_lanczos, kSlqMaxSteps);
  (void)ws;
  (void)ws_bytes;
  hipLaunchKernelGGL(slq_probe_kernel, dim3(nprobe), dim3(kSlqThreads), 0, stream, nprobe, n_lanczos, lanczos_ab, iters,
                     bnorm2, contrib);
  GPL_LAUNCH_CHECK();
  hipLaunchKernelGGL(slq_sum_kernel, dim3(1), dim3(64), 0, stream, nprobe, scale, offset, contrib, logdet,
                     stderr_out);
  GPL_LAUNCH_CHECK();
  return GPL_OK;
}
