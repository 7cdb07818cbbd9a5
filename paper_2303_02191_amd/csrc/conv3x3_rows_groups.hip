// The pipelined 3x3 kernel (rows_kernel.h) for layout 1, three groups of taps without a centre: its stage is RowSchedule's neighbour
// GroupSchedule there.  A file of its own because each layout's kernels take minutes to compile.
#include "rows_kernel.h"

namespace rtoss {

rtoss_status launch_conv3x3_rows_groups(const rtoss_wdesc& d, const ConvParams& c, const RowsLaunch* planned, const void* section, const void* x,
                                        void* y, hipStream_t s)
{
    return launch_rows_typed<1>(d, c, planned, section, x, y, s);
}

}  // namespace rtoss
