// All-float32 spectral pipelines, half-lengths up to kNhLoMax.
#include "pipeline_run.h"

namespace llg {
LLG_PIPELINE_PART(float, float, float, false)
}  // namespace llg
