// All-float32 spectral pipelines.
#include "pipeline_run.h"

namespace llg {
template hipError_t run_pipeline<float, float, float>(const Ctx&, int, int, const SymArgs&, const NodalArgs&,
                                                      const PipeIO<float, float, float>&, hipStream_t,
                                                         const BasisDots*, double*);
}  // namespace llg
