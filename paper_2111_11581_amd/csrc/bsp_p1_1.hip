// Instantiations of the kernel of bf16 pointwise layers: stride 1.
#include "bsp_p1.h"

namespace bsp {
namespace p1 {

p1_fn pick_1(int NT, int TM, int TPG, bool map, bool ident) {
    return NT == 2 ? p1_pick<1, 2>(TM, TPG, map, ident) : NT == 4 ? p1_pick<1, 4>(TM, TPG, map, ident)
           : NT == 8 ? p1_pick<1, 8>(TM, TPG, map, ident) : nullptr;
}

}  // namespace p1
}  // namespace bsp
