// tau1_lines.hip -- the row kernels of one precision (TAU1_P from the build):
// every 3-D lattice, rows of any length.
#include "tau1_lines.hpp"

#ifndef TAU1_P
#error "TAU1_P must be set by the build"
#endif

#define TAU1_CAT2(a, b) a##b
#define TAU1_CAT(a, b) TAU1_CAT2(a, b)

namespace tau1 {

void* TAU1_CAT(ln_kernel_, TAU1_P)(int q) {
    switch (q) {
        case 15: return reinterpret_cast<void*>(&k_lines<15, TAU1_P>);
        case 19: return reinterpret_cast<void*>(&k_lines<19, TAU1_P>);
        case 27: return reinterpret_cast<void*>(&k_lines<27, TAU1_P>);
    }
    return nullptr;
}

}  // namespace tau1
