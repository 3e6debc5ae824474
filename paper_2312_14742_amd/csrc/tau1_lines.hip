// tau1_lines.hip -- the kernels for rows of any length in one precision (TAU1_P
// from the build), every 3-D lattice: one node per lane, and for rows of a few
// nodes one per thread.
#include "tau1_nodes.hpp"

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

void* TAU1_CAT(nd_kernel_, TAU1_P)(int q) {
    switch (q) {
        case 15: return reinterpret_cast<void*>(&k_nodes<15, TAU1_P>);
        case 19: return reinterpret_cast<void*>(&k_nodes<19, TAU1_P>);
        case 27: return reinterpret_cast<void*>(&k_nodes<27, TAU1_P>);
    }
    return nullptr;
}

}  // namespace tau1
