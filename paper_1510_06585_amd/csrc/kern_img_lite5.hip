// Stencil image kernels with a histogram: value stages solarise, noise and noise, solarise before the blur, up to two after it.
#include "kern_img_dev.h"

namespace skel {

static const ImgEntry kTable[] = {
    SKEL_IMG_LITE(6, 0, true, true, "img_chain_blur_reduce"),
    SKEL_IMG_LITE_PRE(6, true, "img_chain_blur_reduce"),
    SKEL_IMG_LITE_PRE(9, true, "img_chain_blur_reduce"),
};

ImgEntries img_lite_5() { return {kTable, (int)(sizeof(kTable) / sizeof(kTable[0]))}; }

}  // namespace skel
