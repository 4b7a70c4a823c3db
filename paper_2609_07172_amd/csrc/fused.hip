// Fused streaming multigrid passes, FP64: the entry points of the V-cycle and
// the passes of the default sweep counts (the pass itself is in fused_pass.h).
#include "fused_pass.h"

namespace cp {

bool fused_supported(const cylpoisson_plan* p, int l) {
    if (!p->opt.fused || p->opt.smoother != 0 || l + 1 >= (int)p->dl.size()) return false;
    const int n1 = nu_pre(p, l), n2 = nu_post(p, l);
    if (n1 > 4 || n2 > 4) return false;
    // 32-bit offsets within a chunk's rows and within a coarse plane
    const LevelView& v = p->dl[l].v;
    const LevelView& vc = p->dl[l + 1].v;
    const Shape sd = pass_shape<double>(p, l, n1, true), su = pass_shape<double>(p, l, n2, false);
    const long long rows = std::max(sd.chunk, su.chunk) + 64;
    return std::max(sd.nstrips, su.nstrips) <= kSlotPartial && rows * v.pitch * 8 < kMaxRange &&
           (long long)vc.nz * vc.pitch * 8 < kMaxRange;
}

namespace {

// A pass of the default sweep count by the level's coefficients; other counts
// are compiled in fused_nu.hip.
template <int KIND>
hipError_t launch_pass(int nu, bool fine, const Shape& sh, const PassArgs<double>& a, int np, hipStream_t s) {
    constexpr int kNu = KIND == kMerge ? 4 : 2;
    if (nu != kNu) return launch_other(KIND, nu, fine, sh, a, np, s);
    switch (sh.coef) {
        case kOneBand: return launch_zc<double, kNu, KIND, kOneBand>(fine, sh, a, np, s);
        case kSomeRows:
            if constexpr (KIND != kMerge) return launch_zc<double, kNu, KIND, kSomeRows>(fine, sh, a, np, s);
            return hipErrorInvalidValue;
        default: return launch_zc<double, kNu, KIND, kRowTables>(fine, sh, a, np, s);
    }
}

}  // namespace

hipError_t fused_down(cylpoisson_plan* p, int l, bool zero_u, bool zero_interior, hipStream_t s,
                      int p0, int np) {
    if (np < 0) np = p->nt;
    DeviceLevel& L = p->dl[l];
    DeviceLevel& C = p->dl[l + 1];
    const int nu = nu_pre(p, l);
    const Shape sh = pass_shape<double>(p, l, nu, true);
    PassArgs<double> a = make_args<double>(p, l, sh, p0, np);
    a.u_in = L.u;
    a.f = L.f;
    a.u_out = L.u2;
    a.fc = C.f;
    if (zero_u) return launch_pass<kDownZero>(nu, l == 0, sh, a, np, s);
    if (zero_interior) return launch_pass<kDownRing>(nu, l == 0, sh, a, np, s);
    return launch_pass<kDownFull>(nu, l == 0, sh, a, np, s);
}

// The first down pass on level l after a full-multigrid start, with the
// start's interpolation from level l + 1 folded in: two or three pre-sweeps,
// fused passes on level l.  The finest level's first cycle uses it, and so
// does the start's own V-cycle on level 1.  With "prefetch" 2 or 3 the start is
// written out and read back instead, which a plan can compare this with.
bool fused_down_pro_ok(const cylpoisson_plan* p, int l) {
    const int nu = nu_pre(p, l);
    return fused_supported(p, l) && (nu == 2 || nu == 3) && p->opt.prefetch == 1;
}

hipError_t fused_down_pro(cylpoisson_plan* p, hipStream_t s, int p0, int np, int l) {
    if (np < 0) np = p->nt;
    DeviceLevel& L = p->dl[l];
    DeviceLevel& C = p->dl[l + 1];
    const int nu = nu_pre(p, l);
    const Shape sh = pass_shape<double>(p, l, nu, true);
    PassArgs<double> a = make_args<double>(p, l, sh, p0, np);
    a.u_in = L.u;  // its ring; the interior is zero plus the prolongated C.u
    a.f = L.f;
    a.u_out = L.u2;
    a.fc = C.f;
    a.ec = C.u;
    return launch_pass<kDownPro>(nu, l == 0, sh, a, np, s);
}

// The merged finest pass: nu2 sweeps after one finest coarse-grid correction
// and nu1 before the next (4 to 6 in a row), fused passes on the finest level,
// at most 513 radial nodes.
bool fused_merge_ok(const cylpoisson_plan* p) {
    const int nu = nu_pre(p, 0) + nu_post(p, 0);
    return p->opt.merge && fused_supported(p, 0) && nu >= 4 && nu <= 6 && p->nr <= 513;
}

hipError_t fused_merge(cylpoisson_plan* p, hipStream_t s) {
    DeviceLevel& L = p->dl[0];
    DeviceLevel& C = p->dl[1];
    const int nu = nu_pre(p, 0) + nu_post(p, 0);
    const Shape sh = pass_shape<double>(p, 0, nu, true, true);
    PassArgs<double> a = make_args<double>(p, 0, sh, 0, p->nt);
    a.u_in = L.u2;  // the last down pass's iterate, plus the prolongated C.u
    a.f = L.f;
    a.u_out = L.u;
    a.fc = C.f;
    a.ec = C.u;
    return launch_pass<kMerge>(nu, true, sh, a, p->nt, s);
}

int fused_chunks(const cylpoisson_plan* p, int l, int nu) {
    return pass_shape<double>(p, l, nu, false).per_plane;
}

hipError_t fused_up(cylpoisson_plan* p, int l, double* partial, int partial_ld, int* npartial,
                    hipStream_t s, int p0, int np) {
    if (np < 0) np = p->nt;
    DeviceLevel& L = p->dl[l];
    DeviceLevel& C = p->dl[l + 1];
    const int nu = nu_post(p, l);
    const Shape sh = pass_shape<double>(p, l, nu, false);
    PassArgs<double> a = make_args<double>(p, l, sh, p0, np);
    a.u_in = L.u2;
    a.f = L.f;
    a.u_out = L.u;
    a.ec = C.u;
    a.partial = partial;
    a.partial_ld = partial_ld;
    if (npartial) *npartial = sh.per_plane;
    return launch_pass<kUp>(nu, l == 0, sh, a, np, s);
}

}  // namespace cp
