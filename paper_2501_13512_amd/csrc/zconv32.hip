#include "zconv.h"

namespace vie {
template void launch_zconv<float>(int, const ZArgs<float>&, int, hipStream_t);
}  // namespace vie
