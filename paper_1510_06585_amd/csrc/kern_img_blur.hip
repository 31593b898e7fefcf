// Image kernels with a stencil (9 = noise then solarise before it).
#include "kern_img_dev.h"

namespace skel {

static const ImgEntry kTable[] = {
    SKEL_IMG_STENCIL(0, false, "img_blur"),
    SKEL_IMG_STENCIL(9, false, "img_noise_sol_blur"),
};

ImgEntries img_entries_blur() { return {kTable, (int)(sizeof(kTable) / sizeof(kTable[0]))}; }

}  // namespace skel
