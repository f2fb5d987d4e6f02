// kb_f32fb.hip -- the builds in FP32 with the FP64 fallback.
#include "kb_launch.hpp"

namespace kb {
KB_INSTANCES(, Prec::F32FB)
}  // namespace kb
