// xloop_f32.hip -- the XCD-grouped loop's variants for fp32 data, H <= 512.
#include "xloop_kernel.h"
namespace ldyn {
extern const XVariant kXF32[];
const XVariant kXF32[] = {
    XV_NT(0, EltF32, 1, 4, 4),  XV_NT(0, EltF32, 1, 8, 4),  XV_NT(0, EltF32, 2, 16, 4),
    XV_NT(0, EltF32, 3, 24, 4), XV_NT(0, EltF32, 4, 32, 4),
    XVariant{},
};
}  // namespace ldyn
