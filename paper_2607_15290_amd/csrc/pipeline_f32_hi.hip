// All-float32 spectral pipelines, half-lengths above kNhLoMax.
#include "pipeline_run.h"

namespace llg {
LLG_PIPELINE_PART(float, float, float, true)
}  // namespace llg
