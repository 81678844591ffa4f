// Eq. (2) on the device: the reference fingerprint from L images and their noise
// residuals.
#include "kernels.hpp"

namespace prnu {

namespace {

// Eq. (2): reference fingerprint K = sum_l I_l W_l / sum_l I_l^2, pixel-wise, with FP64
// accumulators.  Each thread owns four consecutive pixels and streams the L images and
// residuals once; zero where the images are dark.  Bound by memory.
// With an M N that is no multiple of 4 the images lie 4-byte aligned only; the same
// 16-byte loads then ask for no more than that (32 images of 1079 x 1921: a call 147 us,
// against 410 with a thread's four pixels summed one after the other from 4-byte loads).

typedef float Quad __attribute__((ext_vector_type(4)));
typedef float Quad4 __attribute__((ext_vector_type(4), aligned(4)));

template <class V, bool NT>
__device__ __forceinline__ V load_quad(const float* p) {
  if constexpr (NT)
    return __builtin_nontemporal_load(reinterpret_cast<const V*>(p));
  else
    return *reinterpret_cast<const V*>(p);
}

template <class V, bool NT>
__device__ __forceinline__ void estimate_quad(const float* __restrict__ I, const float* __restrict__ W, int L,
                                              int64_t MN, int64_t p0, float* __restrict__ K) {
  double n[4] = {0.0, 0.0, 0.0, 0.0}, d[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
  for (int l = 0; l < L; ++l) {
    const V i = load_quad<V, NT>(I + (int64_t)l * MN + p0);
    const V w = load_quad<V, NT>(W + (int64_t)l * MN + p0);
    n[0] = fma((double)i.x, (double)w.x, n[0]);
    n[1] = fma((double)i.y, (double)w.y, n[1]);
    n[2] = fma((double)i.z, (double)w.z, n[2]);
    n[3] = fma((double)i.w, (double)w.w, n[3]);
    d[0] = fma((double)i.x, (double)i.x, d[0]);
    d[1] = fma((double)i.y, (double)i.y, d[1]);
    d[2] = fma((double)i.z, (double)i.z, d[2]);
    d[3] = fma((double)i.w, (double)i.w, d[3]);
  }
  float4 k;
  k.x = d[0] > 0.0 ? (float)(n[0] / d[0]) : 0.f;
  k.y = d[1] > 0.0 ? (float)(n[1] / d[1]) : 0.f;
  k.z = d[2] > 0.0 ? (float)(n[2] / d[2]) : 0.f;
  k.w = d[3] > 0.0 ? (float)(n[3] / d[3]) : 0.f;
  *reinterpret_cast<float4*>(K + p0) = k;
}

template <int T, bool NT>
__global__ __launch_bounds__(T) void k_estimate_fp(const float* __restrict__ I, const float* __restrict__ W,
                                                   int L, int64_t MN, float* __restrict__ K) {
  const int64_t p0 = ((int64_t)blockIdx.x * T + threadIdx.x) * 4;
  if (p0 >= MN) return;
  if ((MN & 3) == 0) {  // every image's fours are 16-byte aligned, like the buffers
    estimate_quad<Quad, NT>(I, W, L, MN, p0, K);
  } else if (p0 + 4 <= MN) {
    estimate_quad<Quad4, NT>(I, W, L, MN, p0, K);
  } else {
    for (int64_t p = p0; p < MN; ++p) {
      double nn = 0.0, dd = 0.0;
      for (int l = 0; l < L; ++l) {
        const double i = I[(int64_t)l * MN + p], w = W[(int64_t)l * MN + p];
        nn = fma(i, w, nn);
        dd = fma(i, i, dd);
      }
      K[p] = dd > 0.0 ? (float)(nn / dd) : 0.f;
    }
  }
}

}  // namespace

hipError_t launch_estimate_fp(const float* I, const float* W, int L, int64_t MN, float* K, hipStream_t s) {
  if (MN <= 0) return hipSuccess;
  const int64_t threads = (MN + 3) / 4;
  const dim3 grid((unsigned)((threads + 255) / 256));
  // Inputs past the 256 MB last-level cache are read past it: 32 images of 1080 x 1920
  // (531 MB) in 88 us, 6.0 TB/s, against 100; 8 of them (133 MB), which a producer may
  // have left there, cost 1 us more that way.
  if (8.0 * L * (double)MN > 256e6)
    k_estimate_fp<256, true><<<grid, 256, 0, s>>>(I, W, L, MN, K);
  else
    k_estimate_fp<256, false><<<grid, 256, 0, s>>>(I, W, L, MN, K);
  return hipGetLastError();
}

}  // namespace prnu
