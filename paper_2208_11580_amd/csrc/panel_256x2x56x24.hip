// Panel kernel variant: 256 threads, 2 owned indices per thread, blocks of 80 steps
// (56 block vectors in registers, 24 in LDS).
#include "panel_impl.h"

namespace obc_blocked {
OBC_DEFINE_PANEL(launch_panel, false, 256, 2, 56, 24)
}
