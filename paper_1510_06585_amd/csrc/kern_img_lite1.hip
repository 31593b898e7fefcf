// Stencil image kernels: value stages solarise and noise twice before the blur, up to two after it.
#include "kern_img_dev.h"

namespace skel {

static const ImgEntry kTable[] = {
    SKEL_IMG_LITE(2, 0, true, false, "img_chain_blur"),
    SKEL_IMG_LITE_PRE(2, false, "img_chain_blur"),
    SKEL_IMG_LITE(5, 0, true, false, "img_chain_blur"),
    SKEL_IMG_LITE_PRE(5, false, "img_chain_blur"),
};

ImgEntries img_lite_1() { return {kTable, (int)(sizeof(kTable) / sizeof(kTable[0]))}; }

}  // namespace skel
