// Symmetric order-4 adjoint product instantiated for one precision; see adjoint_sym.h.
#include "adjoint_sym.h"

namespace ps {

template hipError_t launch_adjoint4_sym_prec<kBF16>(const float*, const uint4*, const float2*, const int*, int,
                                                    long long, float*, cplx<float>*, const cplx<float>*, Geom, int,
                                                    hipStream_t);

}  // namespace ps
