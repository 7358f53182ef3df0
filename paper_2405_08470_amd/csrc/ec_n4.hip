// Instantiations of the elementwise kernel for 4-mode tensors (one
// translation unit per mode count, so they compile in parallel).
#include "ec_kernel.hpp"

namespace spt {

EcFnPtr pick_ec_n4(int rank, int fdtype, int words, int kind, EcForm form, int steps) {
    return pick_layout<4>(rank, fdtype, words, kind, form, steps);
}

}  // namespace spt
