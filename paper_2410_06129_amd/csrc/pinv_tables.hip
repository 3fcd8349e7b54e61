// Encoding tables on the device (Eq. 2): the phase factors of every sample from
// the trajectory, sample times and species frequencies, in FP64 and, for plans
// that need them, rounded to FP32 beside the coil and off-resonance maps.
#include "pinv_internal.h"

namespace pinv {

// exp(-i 2 pi turns), the turn count reduced to [-1/2, 1/2] first (exact; the
// products that form it are rounded, not fused into the reduction).
__device__ __forceinline__ cx<double> phasor(double turns) {
  double s, c;
  sincospi(2.0 * (turns - rint(turns)), &s, &c);
  return cx<double>{c, -s};
}

// One phase factor or map value per thread: first Px, then Py, Q, and (with
// FP32 tables) the coil, b0 and t values to round.  K (nx + ny + S) sincospi in
// FP64: 26 us at 128 x 128 and K = 32768, where one host core took 130 ms and the
// upload of both tables 6 ms.
__global__ __launch_bounds__(256) void k_tables(EncDev<double> e, EncDev<float> f, bool f32,
                                                const double* __restrict__ k,
                                                const double* __restrict__ hz) {
  const int64_t npx = (int64_t)e.K * e.nx, npy = (int64_t)e.K * e.ny, nq = e.q ? (int64_t)e.K * e.S : 0;
  const int64_t nc = e.coil ? 2 * (int64_t)e.C * e.V : 0, nb = e.b0 ? e.V : 0, nt = e.b0 ? e.K : 0;
  const int64_t total = npx + npy + nq + (f32 ? nc + nb + nt : 0);
  for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < total;
       u += (int64_t)gridDim.x * blockDim.x) {
    int64_t j = u;
    if (j < npx + npy + nq) {
      const double *tab64;
      const float* tab32;
      double turns;
      if (j < npx) {
        const int i = (int)(j / e.nx), ix = (int)(j - (int64_t)i * e.nx);
        turns = __dmul_rn(k[2 * i], (ix - e.nx / 2.0) / e.nx);
        tab64 = e.px, tab32 = f.px;
      } else if ((j -= npx) < npy) {
        const int i = (int)(j / e.ny), iy = (int)(j - (int64_t)i * e.ny);
        turns = __dmul_rn(k[2 * i + 1], (iy - e.ny / 2.0) / e.ny);
        tab64 = e.py, tab32 = f.py;
      } else {
        j -= npy;
        const int i = (int)(j / e.S), s = (int)(j - (int64_t)i * e.S);
        turns = __dmul_rn(hz ? hz[s] : 0.0, e.t[i]);
        tab64 = e.q, tab32 = f.q;
      }
      const cx<double> z = phasor(turns);
      reinterpret_cast<cx<double>*>(const_cast<double*>(tab64))[j] = z;
      if (f32)
        reinterpret_cast<cx<float>*>(const_cast<float*>(tab32))[j] = cx<float>{(float)z.re, (float)z.im};
      continue;
    }
    j -= npx + npy + nq;
    if (j < nc) const_cast<float*>(f.coil)[j] = (float)e.coil[j];
    else if ((j -= nc) < nb) const_cast<float*>(f.b0)[j] = (float)e.b0[j];
    else const_cast<float*>(f.t)[j - nb] = (float)e.t[j - nb];
  }
}

hipError_t launch_tables(const EncDev<double>& e, const EncDev<float>* f, const double* k,
                         const double* hz, hipStream_t s) {
  const int64_t n = (int64_t)e.K * (e.nx + e.ny + e.S) + 2 * (int64_t)e.C * e.V + e.V + e.K;
  const int blocks = (int)std::min<int64_t>((n + 255) / 256, 1 << 15);
  hipLaunchKernelGGL(k_tables, dim3(blocks), dim3(256), 0, s, e, f ? *f : EncDev<float>{}, f != nullptr, k,
                     hz);
  return hipGetLastError();
}

}  // namespace pinv
