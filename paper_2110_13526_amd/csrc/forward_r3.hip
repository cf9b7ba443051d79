// forward_r3.hip -- the forward projector with 3 detector rows per lane (kct_forward.h).
#include "kct_forward.h"

namespace kct {

KCT_FORWARD_ROWS(3)

}  // namespace kct
