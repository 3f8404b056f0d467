// float64 spectral pipelines, half-lengths up to kNhLoMax.
#include "pipeline_run.h"

namespace llg {
LLG_PIPELINE_PART(double, double, double, false)
}  // namespace llg
