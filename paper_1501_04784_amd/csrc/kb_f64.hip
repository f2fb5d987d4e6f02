// kb_f64.hip -- the builds in FP64.
#include "kb_launch.hpp"

namespace kb {
KB_INSTANCES(, Prec::F64)
}  // namespace kb
