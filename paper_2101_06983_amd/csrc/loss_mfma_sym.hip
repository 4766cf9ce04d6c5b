// The gradient walks of the symmetric forms (grad_walk.h): the symmetric loss, and NT-Xent, which is its dQ role alone.
#include "grad_walk.h"

namespace gc {

template <int D>
__global__ void __launch_bounds__(256) GR_CODE_ALIGN grad_sym_kernel(GradArgs ga) {
  extern __shared__ __attribute__((aligned(16))) unsigned char gsmem[];
  const bool one_exp = __builtin_amdgcn_readfirstlane(*ga.wide) == 0;   // see kWideLse
  const int nQ = ga.obQ * ga.nsq;
  const int id = xcd_task_id();
  if (id < nQ) {
    if (one_exp) grad_body<D, true, true, false, true>(ga, id % ga.obQ, id / ga.obQ, gsmem);
    else grad_body<D, true, true>(ga, id % ga.obQ, id / ga.obQ, gsmem);
  } else {
    const int t = id - nQ;
    if (one_exp) grad_body<D, false, true, false, true>(ga, t % ga.obP, t / ga.obP, gsmem);
    else grad_body<D, false, true>(ga, t % ga.obP, t / ga.obP, gsmem);
  }
}
template <int D>
static hipError_t grad_sym_launch_as(const GradArgs& ga, int nwg, hipStream_t stream) {
  const int smem = GradCfg<D>::SMEM;
  static bool attr_done[64];
  if (hipError_t e = ensure_dyn_lds((const void*)grad_sym_kernel<D>, smem, attr_done); e != hipSuccess) return e;
  grad_sym_kernel<D><<<nwg, 256, smem, stream>>>(ga);
  return hipGetLastError();
}
hipError_t grad_sym_launch(const GradArgs& ga, int d, int nwg, hipStream_t stream) {
  switch (d) {
    case 256: return grad_sym_launch_as<256>(ga, nwg, stream);
    case 384: return grad_sym_launch_as<384>(ga, nwg, stream);
    case 512: return grad_sym_launch_as<512>(ga, nwg, stream);
    case 640: return grad_sym_launch_as<640>(ga, nwg, stream);
    case 768: return grad_sym_launch_as<768>(ga, nwg, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace gc
