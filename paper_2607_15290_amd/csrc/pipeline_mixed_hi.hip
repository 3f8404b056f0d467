// Mixed spectral pipelines of the precision form, half-lengths above kNhLoMax:
// float32 apply of a float64 Krylov vector, float32 matvec producing a float64
// Krylov vector, float32 apply and fused M^{-1} A between float64 Krylov vectors.
#include "pipeline_run.h"

namespace llg {
LLG_PIPELINE_PART(float, double, float, true)
LLG_PIPELINE_PART(float, float, double, true)
LLG_PIPELINE_PART(float, double, double, true)
}  // namespace llg
