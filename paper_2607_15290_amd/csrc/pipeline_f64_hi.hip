// float64 spectral pipelines, half-lengths above kNhLoMax.
#include "pipeline_run.h"

namespace llg {
LLG_PIPELINE_PART(double, double, double, true)
}  // namespace llg
