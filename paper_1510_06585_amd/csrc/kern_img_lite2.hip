// Stencil image kernels: value stages solarise, noise and noise, solarise before the blur, up to two after it.
#include "kern_img_dev.h"

namespace skel {

static const ImgEntry kTable[] = {
    SKEL_IMG_LITE(6, 0, true, false, "img_chain_blur"),
    SKEL_IMG_LITE_PRE(6, false, "img_chain_blur"),
    SKEL_IMG_LITE_PRE(9, false, "img_chain_blur"),
};

ImgEntries img_lite_2() { return {kTable, (int)(sizeof(kTable) / sizeof(kTable[0]))}; }

}  // namespace skel
