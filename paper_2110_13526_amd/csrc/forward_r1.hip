// forward_r1.hip -- the forward projector with 1 detector row per lane (kct_forward.h).
#include "kct_forward.h"

namespace kct {

KCT_FORWARD_ROWS(1)

}  // namespace kct
