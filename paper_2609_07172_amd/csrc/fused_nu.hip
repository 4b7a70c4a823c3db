// Fused streaming multigrid passes, FP64, for sweep counts other than the
// default's (one, three and four sweeps; five and six merged).  One
// instantiation serves every level: rows outside the regular band form their
// coefficients from the tables, on a stretched mesh all of them (400 x 128 x 512
// cells stretched 4:1, V(3,3): 1.32 ms a cycle, 3.2 as one workgroup per plane
// and chunk).
#include "fused_pass.h"

namespace cp {

namespace {

template <int NU>
hipError_t launch_nu(int kind, bool fine, const Shape& sh, const PassArgs<double>& a, int np, hipStream_t s) {
    switch (kind) {
        case kDownZero: return launch_zc<double, NU, kDownZero, kSomeRows>(fine, sh, a, np, s);
        case kDownRing: return launch_zc<double, NU, kDownRing, kSomeRows>(fine, sh, a, np, s);
        case kDownFull: return launch_zc<double, NU, kDownFull, kSomeRows>(fine, sh, a, np, s);
        case kUp: return launch_zc<double, NU, kUp, kSomeRows>(fine, sh, a, np, s);
        case kDownPro:
            if constexpr (NU == 3) return launch_zc<double, NU, kDownPro, kSomeRows>(fine, sh, a, np, s);
            break;
        default: break;
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_other(int kind, int nu, bool fine, const Shape& sh, const PassArgs<double>& a, int np, hipStream_t s) {
    if (kind == kMerge)
        return nu == 5   ? launch_zc<double, 5, kMerge, kSomeRows>(fine, sh, a, np, s)
               : nu == 6 ? launch_zc<double, 6, kMerge, kSomeRows>(fine, sh, a, np, s)
                         : hipErrorInvalidValue;
    switch (nu) {
        case 1: return launch_nu<1>(kind, fine, sh, a, np, s);
        case 3: return launch_nu<3>(kind, fine, sh, a, np, s);
        case 4: return launch_nu<4>(kind, fine, sh, a, np, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace cp
