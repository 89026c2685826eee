// Symmetric order-3 adjoint product instantiated for one precision; see adjoint_sym.h.
#include "adjoint_sym.h"

namespace ps {

template hipError_t launch_adjoint_sym_prec<kFP32>(const float*, const uint4*, const float2*, int, int,
                                                   long long, float*, cplx<float>*, const cplx<float>*, Geom, int,
                                                   hipStream_t);

}  // namespace ps
