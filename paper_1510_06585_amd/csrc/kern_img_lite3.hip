// Stencil image kernels with a histogram: value stages (none) and noise before the blur, up to two after it.
#include "kern_img_dev.h"

namespace skel {

static const ImgEntry kTable[] = {
    SKEL_IMG_LITE_PRE(0, true, "img_chain_blur_reduce"),
    SKEL_IMG_LITE(1, 0, true, true, "img_chain_blur_reduce"),
    SKEL_IMG_LITE_PRE(1, true, "img_chain_blur_reduce"),
};

ImgEntries img_lite_3() { return {kTable, (int)(sizeof(kTable) / sizeof(kTable[0]))}; }

}  // namespace skel
