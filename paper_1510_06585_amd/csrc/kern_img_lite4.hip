// Stencil image kernels with a histogram: value stages solarise and noise twice before the blur, up to two after it.
#include "kern_img_dev.h"

namespace skel {

static const ImgEntry kTable[] = {
    SKEL_IMG_LITE(2, 0, true, true, "img_chain_blur_reduce"),
    SKEL_IMG_LITE_PRE(2, true, "img_chain_blur_reduce"),
    SKEL_IMG_LITE(5, 0, true, true, "img_chain_blur_reduce"),
    SKEL_IMG_LITE_PRE(5, true, "img_chain_blur_reduce"),
};

ImgEntries img_lite_4() { return {kTable, (int)(sizeof(kTable) / sizeof(kTable[0]))}; }

}  // namespace skel
