#include "frame64.h"

namespace nqs {
namespace frame {

void launch_ln32(const nqs_ctx *c, const FrameArgs &a, int mode, int64_t items, int shape, hipStream_t s)
{
    launch_c<double, 32, kNetLnCosh>(c, a, mode, items, shape, s);
}

}  // namespace frame
}  // namespace nqs
