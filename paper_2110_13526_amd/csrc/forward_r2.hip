// forward_r2.hip -- the forward projector with 2 detector rows per lane (kct_forward.h).
#include "kct_forward.h"

namespace kct {

KCT_FORWARD_ROWS(2)

}  // namespace kct
