#include "frame64.h"

namespace nqs {
namespace frame {

void launch_cnn1(const nqs_ctx *c, const FrameArgs &a, int mode, int64_t items, int shape, hipStream_t s)
{
    launch_c<double, 16, kNetCnn1>(c, a, mode, items, shape, s);
}

}  // namespace frame
}  // namespace nqs
