// Image kernels without a stencil (1 = noise, 2 = solarise, 9 = noise then solarise).
#include "kern_img_dev.h"

namespace skel {

static const ImgEntry kTable[] = {
    SKEL_IMG_POINT(0, false, "img_copy"),
    SKEL_IMG_POINT(1, false, "img_noise"),
    SKEL_IMG_POINT(2, false, "img_solarise"),
    SKEL_IMG_POINT(0, true, "img_reduce"),
    SKEL_IMG_POINT(9, false, "img_noise_sol"),
    SKEL_IMG_POINT(9, true, "img_noise_sol_reduce"),
};

ImgEntries img_entries_point() { return {kTable, (int)(sizeof(kTable) / sizeof(kTable[0]))}; }

}  // namespace skel
