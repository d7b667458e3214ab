// xbwd_f32.hip -- the XCD-grouped reverse loop's variants for fp32 data.
#include "xbwd_kernel.h"
namespace ldyn {
extern const XBVariant kXBF32[];
const XBVariant kXBF32[] = {
    XBV_NT(0, EltF32, 1, 16), XBV_NT(0, EltF32, 1, 32), XBV_NT(0, EltF32, 1, 64),
    XBVariant{},
};
}  // namespace ldyn
