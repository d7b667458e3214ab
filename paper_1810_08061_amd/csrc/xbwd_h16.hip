// xbwd_h16.hip -- the XCD-grouped reverse loop's variants for bf16 data.
#include "xbwd_kernel.h"
namespace ldyn {
extern const XBVariant kXBH16[];
const XBVariant kXBH16[] = {
    XBV_NT(1, EltH16, 1, 2), XBV_NT(1, EltH16, 1, 4), XBV_NT(1, EltH16, 1, 8), XBV_NT(1, EltH16, 2, 16),
    XBVariant{},
};
}  // namespace ldyn
