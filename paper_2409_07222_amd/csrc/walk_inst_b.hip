// Instantiations of the first-step walker for KH in 6..8.
#include "walk_impl.h"

namespace labsdev {

namespace {
template <int KH, int NT, int NQ>
void fill(WalkKernels* o) {
    o->plain = walkimpl::k_walk<KH, NT, NQ>;
    o->bloom = walkimpl::k_walk_bloom<KH, NT, NQ>;
    o->log = walkimpl::k_walk_log<KH, NT, NQ>;
    o->persistent = walkimpl::k_walk_persistent<KH, NT, NQ>;
}
}  // namespace

bool walk_kernels_b(int KH, WalkKernels* o) {
    switch (KH) {
        case 6: fill<6, 1, 1>(o); return true;
        case 7: fill<7, 1, 1>(o); return true;
        case 8: fill<8, 1, 1>(o); return true;
        default: return false;
    }
}

}  // namespace labsdev
