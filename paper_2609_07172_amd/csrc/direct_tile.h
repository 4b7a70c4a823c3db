// The eliminations of the exact coarse solve (see direct.hip), shared by the
// kernels that run them.
#pragma once

#include "cp_internal.h"

namespace cp {

namespace {

typedef double dbl4 __attribute__((ext_vector_type(4)));

constexpr int kSegRows = 4;  // rows of an elimination segment (one lane)

__device__ __forceinline__ int mode_of(int plane, int nc) { return plane < nc ? plane : plane - nc + 1; }

// The elimination factors and radial couplings of a lane's four rows.
struct SegTables {
    double m[kSegRows], rw[kSegRows], re[kSegRows];
    __device__ __forceinline__ void load(const LevelView& v, const double* M, int stride, int seg) {
        const int nri = v.nr - 2;
#pragma unroll
        for (int u = 0; u < kSegRows; ++u) {
            const int i = seg * kSegRows + u;
            m[u] = M[(size_t)u * stride];
            rw[u] = i < nri ? v.rw[i + 1] : 0.0;
            re[u] = i < nri ? v.re[i + 1] : 0.0;
        }
    }
};

// Both recurrences of a lane's segment: g in, w out.  NSEG lanes of a
// wavefront hold the segments of one eigenvector, in order.
template <int NSEG>
__device__ __forceinline__ void eliminate(const SegTables& tb, double (&g)[kSegRows], int seg) {
    double q[kSegRows];
    {
        double d = 0.0, P = 1.0;
#pragma unroll
        for (int u = 0; u < kSegRows; ++u) {
            q[u] = tb.rw[u] * tb.m[u];
            g[u] *= tb.m[u];
            d = fma(q[u], d, g[u]);
            P *= q[u];
        }
#pragma unroll
        for (int o = 1; o < NSEG; o <<= 1) {
            const double Pp = __shfl_up(P, o, NSEG), dp = __shfl_up(d, o, NSEG);
            if (seg >= o) {
                d = fma(P, dp, d);
                P *= Pp;
            }
        }
        double c = __shfl_up(d, 1, NSEG);
        if (seg == 0) c = 0.0;
#pragma unroll
        for (int u = 0; u < kSegRows; ++u) {
            c = fma(q[u], c, g[u]);
            g[u] = c;
        }
    }
    {
        double w = 0.0, P = 1.0;
#pragma unroll
        for (int u = kSegRows - 1; u >= 0; --u) {
            q[u] = tb.re[u] * tb.m[u];
            w = fma(q[u], w, g[u]);
            P *= q[u];
        }
#pragma unroll
        for (int o = 1; o < NSEG; o <<= 1) {
            const double Pp = __shfl_down(P, o, NSEG), wp = __shfl_down(w, o, NSEG);
            if (seg + o < NSEG) {
                w = fma(P, wp, w);
                P *= Pp;
            }
        }
        double c = __shfl_down(w, 1, NSEG);
        if (seg == NSEG - 1) c = 0.0;
#pragma unroll
        for (int u = kSegRows - 1; u >= 0; --u) {
            c = fma(q[u], c, g[u]);
            g[u] = c;
        }
    }
}

}  // namespace

}  // namespace cp
