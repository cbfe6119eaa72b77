// Instantiations of the first-step walker for KH in 9..11.
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

bool walk_kernels_c(int KH, int NT, int NQ, WalkKernels* o) {
    if (KH == 9 && NQ == 1) {
        if (NT == 1) fill<9, 1, 1>(o); else fill<9, 2, 1>(o);
        return true;
    }
    if (KH == 9 && NQ == 2) {
        if (NT == 1) fill<9, 1, 2>(o); else fill<9, 2, 2>(o);
        return true;
    }
    if (KH == 10 && NQ == 2) {
        if (NT == 1) fill<10, 1, 2>(o); else fill<10, 2, 2>(o);
        return true;
    }
    if (KH == 11 && NQ == 2) {
        if (NT == 1) fill<11, 1, 2>(o); else fill<11, 2, 2>(o);
        return true;
    }
    return false;
}

}  // namespace labsdev
