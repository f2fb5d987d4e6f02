// kb_f32.hip -- the builds in FP32.
#include "kb_launch.hpp"

namespace kb {
KB_INSTANCES(, Prec::F32)
}  // namespace kb
