// Image kernels with a stencil and a histogram (9 = noise then solarise before it).
#include "kern_img_dev.h"

namespace skel {

static const ImgEntry kTable[] = {
    SKEL_IMG_STENCIL(0, true, "img_blur_reduce"),
    SKEL_IMG_STENCIL(9, true, "img_noise_sol_blur_reduce"),
};

ImgEntries img_entries_blur_hist() { return {kTable, (int)(sizeof(kTable) / sizeof(kTable[0]))}; }

}  // namespace skel
