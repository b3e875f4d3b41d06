// Instances of the split-operand GETT kernels (gett_split_device.h) with element-wise loads, for any layout and alignment.
#include "gett_split_device.h"

namespace mera {

void launch_gett_split_scalar(const GettArgs& a, int groups, int splits, hipStream_t s, bool akf, bool bkf, int bm, int bn,
     int planes) {
  launch_split<false>(a, groups, splits, s, akf, bkf, bm, bn, planes);
}

}  // namespace mera
