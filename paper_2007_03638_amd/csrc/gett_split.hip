// Instances of the split-operand GETT kernels (gett_split_device.h) with 16-byte loads.
#include "gett_split_device.h"

namespace mera {

void launch_gett_split(const GettArgs& a, int groups, int splits, hipStream_t s, bool akf, bool bkf, int bm, int bn,
     int planes) {
  launch_split<true>(a, groups, splits, s, akf, bkf, bm, bn, planes);
}

}  // namespace mera
