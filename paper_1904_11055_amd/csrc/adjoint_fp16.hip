// Order-3 adjoint product of the FP16 split; see adjoint.h.
#include "adjoint.h"

namespace ps {

hipError_t launch_adjoint_gemm_fp16(const float* D, const uint4* W, const int* vmask, const unsigned* absmax,
                                    const unsigned long long* rowmax, int n_shells, long long G, float* A,
                                    cplx<float>* H2, const cplx<float>* tw, Geom g, int batch, hipStream_t st) {
  dim3 grid((unsigned)(G / kAdjPts), batch);
#define L2(NF, MBN) hipLaunchKernelGGL((adjoint_gemm<NF, MBN>), grid, dim3(kAdjThreads), 0, st, D, W, vmask, \
                                       absmax, rowmax, n_shells, G, A, H2, tw, g)
#define L(NF) do { if (n_shells > 32) L2(NF, 2); else L2(NF, 1); } while (0)
  switch (g.N) {
    case 32: L(32); break;
    case 64: L(64); break;
    case 128: L(128); break;
    case 256: L(256); break;
    case 512: L(512); break;
    default: L(0); break;
  }
#undef L
#undef L2
  return hipGetLastError();
}

}  // namespace ps
