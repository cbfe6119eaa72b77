// Instantiations of the first-step walker for KH in 2..5.
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

bool walk_kernels_a(int KH, WalkKernels* o) {
    switch (KH) {
        case 2: fill<2, 1, 1>(o); return true;
        case 3: fill<3, 1, 1>(o); return true;
        case 4: fill<4, 1, 1>(o); return true;
        case 5: fill<5, 1, 1>(o); return true;
        default: return false;
    }
}

}  // namespace labsdev
