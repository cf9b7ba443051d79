// forward_r4.hip -- the forward projector with 4 detector rows per lane (kct_forward.h).
#include "kct_forward.h"

namespace kct {

KCT_FORWARD_ROWS(4)

}  // namespace kct
