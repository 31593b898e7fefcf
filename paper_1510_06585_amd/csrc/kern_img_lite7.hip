// Image kernels with a histogram and without a stencil for the less common value stages.
#include "kern_img_dev.h"

namespace skel {

static const ImgEntry kTable[] = {
    SKEL_IMG_LITE(1, 0, false, true, "img_chain_reduce"),
    SKEL_IMG_LITE(2, 0, false, true, "img_chain_reduce"),
    SKEL_IMG_LITE(5, 0, false, true, "img_chain_reduce"),
    SKEL_IMG_LITE(6, 0, false, true, "img_chain_reduce"),
};

ImgEntries img_lite_7() { return {kTable, (int)(sizeof(kTable) / sizeof(kTable[0]))}; }

}  // namespace skel
