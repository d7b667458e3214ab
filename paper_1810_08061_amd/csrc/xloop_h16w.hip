// xloop_h16w.hip -- the XCD-grouped loop's variants for bf16 data, H 513 to 1024.
#include "xloop_kernel.h"
namespace ldyn {
extern const XVariant kXH16W[];
const XVariant kXH16W[] = {
    XV_NT(1, EltH16, 6, 3, 8), XV_NT(1, EltH16, 8, 4, 8),
    XVariant{},
};
}  // namespace ldyn
