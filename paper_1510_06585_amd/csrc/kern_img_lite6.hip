// Image kernels without a stencil for the less common value stages.
#include "kern_img_dev.h"

namespace skel {

static const ImgEntry kTable[] = {
    SKEL_IMG_LITE(5, 0, false, false, "img_chain"),
    SKEL_IMG_LITE(6, 0, false, false, "img_chain"),
};

ImgEntries img_lite_6() { return {kTable, (int)(sizeof(kTable) / sizeof(kTable[0]))}; }

}  // namespace skel
