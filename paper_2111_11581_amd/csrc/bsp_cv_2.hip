// Instantiations of the kernel of 3-wide bf16 convs: stride 2.
#include "bsp_cv.h"

namespace bsp {
namespace cv {

cv_fn pick_2(int NT, int TM, int TPG, bool map) {
    return NT == 2 ? cv_pick<2, 2>(TM, TPG, map) : NT == 4 ? cv_pick<2, 4>(TM, TPG, map)
           : NT == 8 ? cv_pick<2, 8>(TM, TPG, map) : nullptr;
}

}  // namespace cv
}  // namespace bsp
