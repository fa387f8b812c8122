#include "zconv.h"

namespace vie {
template void launch_zconv<double>(int, const ZArgs<double>&, int, hipStream_t);
}  // namespace vie
