// xloop_h16.hip -- the XCD-grouped loop's variants for bf16 data, H <= 512.
#include "xloop_kernel.h"
namespace ldyn {
extern const XVariant kXH16[];
const XVariant kXH16[] = {
    XV_NT(1, EltH16, 1, 1, 4), XV_NT(1, EltH16, 2, 2, 4), XV_NT(1, EltH16, 3, 3, 4), XV_NT(1, EltH16, 4, 4, 4),
    XVariant{},
};
}  // namespace ldyn
