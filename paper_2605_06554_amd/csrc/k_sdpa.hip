// k_sdpa.hip -- dense causal SDPA on the gathered sub-sequence (Sec. 3.5, Eq. attn-sub with
// Eq. sdpa): dispatch and the Delta = rowsum(dO * O) kernel of the backward. The bf16 kernels are
// in k_sdpa_mfma.hip, the fp32 kernels in k_sdpa_f32.hip.
#include <mutex>

#include "lh_common.h"

hipError_t lh_launch_sdpa_fwd_bf16(const LhShape& s, const void* qs, const void* ks, const void* vs, void* os,
                                   float* lse, hipStream_t st);
hipError_t lh_launch_sdpa_bwd_bf16(const LhShape& s, const void* qs, const void* ks, const void* vs,
                                   const void* dos, const float* lse, const float* delta, void* dqs,
                                   void* dks, void* dvs, hipStream_t st);
hipError_t lh_launch_sdpa_fwd_f32(const LhShape& s, const void* qs, const void* ks, const void* vs, void* os,
                                  float* lse, hipStream_t st);
hipError_t lh_launch_sdpa_bwd_f32(const LhShape& s, const void* qs, const void* ks, const void* vs, const void* dos,
                                  const float* lse, const float* delta, void* dqs, void* dks, void* dvs,
                                  hipStream_t st);
hipError_t lh_launch_sdpa_fwd_idx(const LhShape& s, const void* q, const void* k, const void* v, const void* qp,
                                  const void* kp, const void* vp, const int32_t* idx, void* os, float* lse,
                                  hipStream_t st);
hipError_t lh_launch_sdpa_bwd_idx(const LhShape& s, const void* q, const void* k, const void* v, const void* qp,
                                  const void* kp, const void* vp, const int32_t* idx, const void* dos,
                                  const float* lse, const float* delta, void* dqs, void* dks, void* dvs,
                                  hipStream_t st);

namespace lh {

// ------------------------------------------------------------------ Delta = rowsum(dO * O)
template <typename T>
__global__ void __launch_bounds__(256) sdpa_delta(const T* __restrict__ O, const T* __restrict__ dO,
                                                  float* __restrict__ delta, int64_t rows, int D) {
  constexpr int CH = 16 / sizeof(T);
  const int CPR = D / CH;  // 16 or 8 or 32 threads per row
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t row = t / CPR;
  const int cc = (int)(t % CPR);
  float acc = 0.0f;
  if (row < rows) {
    float a[CH], b[CH];
    load_chunk<T>(O + row * D + cc * CH, a);
    load_chunk<T>(dO + row * D + cc * CH, b);
#pragma unroll
    for (int c = 0; c < CH; ++c) acc += a[c] * b[c];
  }
  for (int d = 1; d < CPR; d <<= 1) acc += __shfl_xor(acc, d, 64);
  if (row < rows && cc == 0) delta[row] = acc;
}

}  // namespace lh

using namespace lh;

hipError_t lh_launch_sdpa_fwd(const LhShape& s, const void* qs, const void* ks, const void* vs,
                              void* os, float* lse, hipStream_t st) {
  if (s.S == 0) return hipSuccess;
  if (s.dtype == LH_BF16) return lh_launch_sdpa_fwd_bf16(s, qs, ks, vs, os, lse, st);
  return lh_launch_sdpa_fwd_f32(s, qs, ks, vs, os, lse, st);
}

static hipError_t launch_delta(const LhShape& s, const void* os, const void* dos, float* delta, hipStream_t st) {
  const int64_t rows = s.B * s.Hq * s.S;
  const int CPR = s.D / (s.dtype == LH_BF16 ? 8 : 4);
  dim3 grid((unsigned)((rows * CPR + 255) / 256));
  if (s.dtype == LH_BF16)
    hipLaunchKernelGGL(sdpa_delta<bf16_t>, grid, dim3(256), 0, st, (const bf16_t*)os, (const bf16_t*)dos, delta, rows, s.D);
  else
    hipLaunchKernelGGL(sdpa_delta<float>, grid, dim3(256), 0, st, (const float*)os, (const float*)dos, delta, rows, s.D);
  return hipGetLastError();
}

hipError_t lh_launch_sdpa_fwd_indexed(const LhShape& s, const void* q, const void* k, const void* v,
                                      const void* qpyr, const void* kpyr, const void* vpyr,
                                      const int32_t* idx, void* os, float* lse, hipStream_t st) {
  if (s.S == 0) return hipSuccess;
  return lh_launch_sdpa_fwd_idx(s, q, k, v, qpyr, kpyr, vpyr, idx, os, lse, st);
}

hipError_t lh_launch_sdpa_bwd_indexed(const LhShape& s, const void* q, const void* k, const void* v,
                                      const void* qpyr, const void* kpyr, const void* vpyr,
                                      const int32_t* idx, const void* os, const float* lse,
                                      const void* dos, void* dqs, void* dks, void* dvs, float* delta,
                                      hipStream_t st) {
  if (s.S == 0) return hipSuccess;
  hipError_t e = launch_delta(s, os, dos, delta, st);
  if (e != hipSuccess) return e;
  return lh_launch_sdpa_bwd_idx(s, q, k, v, qpyr, kpyr, vpyr, idx, dos, lse, delta, dqs, dks, dvs, st);
}

hipError_t lh_launch_sdpa_bwd(const LhShape& s, const void* qs, const void* ks, const void* vs,
                              const void* os, const float* lse, const void* dos, void* dqs,
                              void* dks, void* dvs, float* delta, hipStream_t st) {
  if (s.S == 0) return hipSuccess;
  const hipError_t e = launch_delta(s, os, dos, delta, st);
  if (e != hipSuccess) return e;
  if (s.dtype == LH_BF16) return lh_launch_sdpa_bwd_bf16(s, qs, ks, vs, dos, lse, delta, dqs, dks, dvs, st);
  return lh_launch_sdpa_bwd_f32(s, qs, ks, vs, dos, lse, delta, dqs, dks, dvs, st);
}

// ------------------------------------------------------------------ scratch of lh_sdpa_bwd_noalloc
// Delta of the backward (B * Hq * S floats) for callers that cannot allocate: a file-scope
// device array, one copy per GPU, held until the process ends. Its address on the current
// device is looked up once per device with hipGetSymbolAddress; host code never passes the
// array's name itself to a kernel. sdpa_delta overwrites every element a call reads, so
// nothing needs clearing between calls; calls that overlap on one GPU share the array and race.
static constexpr size_t kSdpaScratchBytes = (size_t)16 << 20;
static constexpr int kMaxDevices = 64;
static __device__ __align__(256) unsigned char scratch[kSdpaScratchBytes];
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[kMaxDevices] = {};

size_t lh_sdpa_scratch_bytes() { return kSdpaScratchBytes; }

hipError_t lh_sdpa_scratch(float** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *out = reinterpret_cast<float*>(g_scratch_ptr[dev]);
  return hipSuccess;
}
