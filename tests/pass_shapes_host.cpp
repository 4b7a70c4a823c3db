// Launch shapes of the fused passes, on the CPU: the form that a shape names is
// one that its sweep count is compiled in, and an automatic shape has at most as
// many wavefronts as that form keeps resident.
#include <cstdio>

#include "fused_pass.h"

using namespace cp;

template <typename T>
int check(const cylpoisson_plan& p, int l, int outside) {
    int bad = 0;
    for (int nu = 1; nu <= 6; ++nu)
        for (int kind = 0; kind < 3; ++kind) {  // up, down, merged
            const bool merge = kind == 2;
            if (merge ? nu < 4 || l > 0 : nu > 4) continue;
            const Shape s = pass_shape<T>(&p, l, nu, kind > 0, merge);
            const bool every_form = nu == (merge ? 4 : 2);
            const int resident = 1024 * pass_waves<T>(nu, s.coef, kind == 1 && l > 0);
            if ((every_form || s.coef == kSomeRows) && (s.per_plane * p.nt <= resident || s.nchunks == 1)) continue;
            std::printf("%d x %d x %d, FP%d level %d, %d rows outside, %d sweeps, kind %d: form %d, %d wavefronts, %d resident\n",
                        p.dl[l].v.nr, p.nt, p.dl[l].v.nz, (int)sizeof(T) * 8, l, outside, nu, kind, s.coef,
                        s.per_plane * p.nt, resident);
            ++bad;
        }
    return bad;
}

int main() {
    int bad = 0;
    const int sizes[][2] = {{129, 129}, {400, 512}, {257, 1000}};
    for (const auto& z : sizes)
        for (int nt : {16, 64, 128})
            for (int outside : {0, 2, 4, 5, z[1] - 2}) {
                cylpoisson_plan p;
                p.nt = nt;
                p.dl.resize(3);
                for (int l = 0; l < 3; ++l) {
                    p.dl[l].v.nr = p.dl[l].v.pitch = ((z[0] - 1) >> l) + 1;
                    p.dl[l].v.nz = ((z[1] - 1) >> l) + 1;
                    p.dl[l].reg_lo = 1;
                    p.dl[l].reg_hi = std::max(1, p.dl[l].v.nz - 1 - outside);
                }
                for (int l = 0; l < 2; ++l) bad += check<double>(p, l, outside) + check<float>(p, l, outside);
            }
    return bad != 0;
}
