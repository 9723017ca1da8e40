// Instantiations of the kernel of 3-wide bf16 convs: stride 1.
#include "bsp_cv.h"

namespace bsp {
namespace cv {

cv_fn pick_1(int NT, int TM, int TPG, bool map) {
    return NT == 2 ? cv_pick<1, 2>(TM, TPG, map) : NT == 4 ? cv_pick<1, 4>(TM, TPG, map)
           : NT == 8 ? cv_pick<1, 8>(TM, TPG, map) : nullptr;
}

}  // namespace cv
}  // namespace bsp
