// Stencil image kernels: value stages (none) and noise before the blur, up to two after it.
#include "kern_img_dev.h"

namespace skel {

static const ImgEntry kTable[] = {
    SKEL_IMG_LITE_PRE(0, false, "img_chain_blur"),
    SKEL_IMG_LITE(1, 0, true, false, "img_chain_blur"),
    SKEL_IMG_LITE_PRE(1, false, "img_chain_blur"),
};

ImgEntries img_lite_0() { return {kTable, (int)(sizeof(kTable) / sizeof(kTable[0]))}; }

}  // namespace skel
