// Image kernels that interpret their stage lists.
#include "kern_img_dev.h"

namespace skel {

static const ImgEntry kTable[] = {
    SKEL_IMG_ENTRY(kGeneric, kGeneric, false, false, -1, "img_generic"),
    SKEL_IMG_ENTRY(kGeneric, kGeneric, false, true, -1, "img_generic_reduce"),
    SKEL_IMG_ENTRY(kGeneric, kGeneric, true, false, -1, "img_generic_blur"),
    SKEL_IMG_ENTRY(kGeneric, kGeneric, true, true, -1, "img_generic_blur_reduce"),
};

ImgEntries img_entries_generic() { return {kTable, (int)(sizeof(kTable) / sizeof(kTable[0]))}; }

}  // namespace skel
