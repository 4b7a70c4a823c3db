// Fused streaming multigrid passes in FP32: the inner V-cycles of the
// mixed-precision solve.  Same pass as the FP64 path (fused_pass.h) on the
// FP32 level buffers.
#include "fused_pass.h"

namespace cp {

namespace {

template <int NU, int KIND>
hipError_t launch32(bool fine, const Shape& sh, const PassArgs<float>& a, int np, hipStream_t s) {
    // the default sweep counts by the level's coefficients; for the others one
    // instantiation serves every level
    if constexpr (NU == 2 || KIND == kMerge) {
        if (sh.coef == kOneBand) return launch_zc<float, NU, KIND, kOneBand>(fine, sh, a, np, s);
        if (sh.coef == kRowTables) return launch_zc<float, NU, KIND, kRowTables>(fine, sh, a, np, s);
    }
    if constexpr (KIND == kMerge)
        return hipErrorInvalidValue;
    else
        return launch_zc<float, NU, KIND, kSomeRows>(fine, sh, a, np, s);
}

template <int KIND>
hipError_t launch_pass(int nu, bool fine, const Shape& sh, const PassArgs<float>& a, int np, hipStream_t s) {
    switch (nu) {
        case 1: return launch32<1, KIND>(fine, sh, a, np, s);
        case 2: return launch32<2, KIND>(fine, sh, a, np, s);
        case 3: return launch32<3, KIND>(fine, sh, a, np, s);
        case 4: return launch32<4, KIND>(fine, sh, a, np, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t fused_down32(cylpoisson_plan* p, int l, bool zero_u, hipStream_t s, int p0, int np) {
    if (np < 0) np = p->nt;
    DeviceLevel32& L = p->dl32[l];
    DeviceLevel32& C = p->dl32[l + 1];
    const int nu = nu_pre(p, l);
    const Shape sh = pass_shape<float>(p, l, nu, true);
    PassArgs<float> a = make_args<float>(p, l, sh, p0, np);
    a.u_in = L.u;
    a.f = L.f;
    a.u_out = L.u2;
    a.fc = C.f;
    return zero_u ? launch_pass<kDownZero>(nu, l == 0, sh, a, np, s) : launch_pass<kDownFull>(nu, l == 0, sh, a, np, s);
}

hipError_t fused_up32(cylpoisson_plan* p, int l, hipStream_t s, int p0, int np) {
    if (np < 0) np = p->nt;
    DeviceLevel32& L = p->dl32[l];
    DeviceLevel32& C = p->dl32[l + 1];
    const int nu = nu_post(p, l);
    const Shape sh = pass_shape<float>(p, l, nu, false);
    PassArgs<float> a = make_args<float>(p, l, sh, p0, np);
    a.u_in = L.u2;
    a.f = L.f;
    a.u_out = L.u;
    a.ec = C.u;
    return launch_pass<kUp>(nu, l == 0, sh, a, np, s);
}

bool fused_merge32_ok(const cylpoisson_plan* p) { return fused_merge_ok(p) && nu_pre(p, 0) + nu_post(p, 0) == 4; }

hipError_t fused_merge32(cylpoisson_plan* p, hipStream_t s) {
    DeviceLevel32& L = p->dl32[0];
    DeviceLevel32& C = p->dl32[1];
    const Shape sh = pass_shape<float>(p, 0, 4, true, true);
    PassArgs<float> a = make_args<float>(p, 0, sh, 0, p->nt);
    a.u_in = L.u2;
    a.f = L.f;
    a.u_out = L.u;
    a.fc = C.f;
    a.ec = C.u;
    return launch32<4, kMerge>(true, sh, a, p->nt, s);
}

}  // namespace cp
