// Order-4 adjoint product of the FP16 split; see adjoint.h.
#include "adjoint.h"

namespace ps {

hipError_t launch_adjoint4_gemm_fp16(const float* D, const uint4* W, const int* imask, const unsigned* absmax,
                                     const unsigned long long* rowmax, int n_shells, long long G, float* A,
                                     cplx<float>* H2, const cplx<float>* tw, Geom g, int batch, hipStream_t st) {
  dim3 grid((unsigned)(G / kAdjPts), batch);
#define L4(NF, NC) hipLaunchKernelGGL((adjoint4_gemm<NF, NC>), grid, dim3(kAdjThreads), 0, st, D, W, imask, \
                                      absmax, rowmax, n_shells, G, A, H2, tw, g)
#define L(NF)                      \
  do {                             \
    if (n_shells <= 32) L4(NF, 2); \
    else L4(NF, 4);                \
  } while (0)
  switch (g.N) {
    case 32: L(32); break;
    case 64: L(64); break;
    case 128: L(128); break;
    case 256: L(256); break;
    case 512: L(512); break;
    default: L(0); break;
  }
#undef L
#undef L4
  return hipGetLastError();
}

}  // namespace ps
