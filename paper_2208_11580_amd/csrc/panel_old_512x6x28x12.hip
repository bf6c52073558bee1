// Panel kernel variant: 512 threads, 6 owned indices per thread, blocks of 40 steps
// (28 block vectors in registers, 12 in LDS), for panels that follow others of their outer block.
#include "panel_impl.h"

namespace obc_blocked {
OBC_DEFINE_PANEL(launch_panel_old, true, 512, 6, 28, 12)
}
