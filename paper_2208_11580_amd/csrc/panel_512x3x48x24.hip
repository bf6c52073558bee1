// Panel kernel variant: 512 threads, 3 owned indices per thread, blocks of 72 steps
// (48 block vectors in registers, 24 in LDS).
#include "panel_impl.h"

namespace obc_blocked {
OBC_DEFINE_PANEL(launch_panel, false, 512, 3, 48, 24)
}
