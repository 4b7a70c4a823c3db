// V-cycles of small planes with everything in one workgroup, for gfx950.
//
// Where level 1 is solved exactly by one workgroup per plane (direct.hip) and
// the finest plane is small, every cycle from one convergence check to the next
// runs in one launch: a workgroup holds its plane's iterate and residual in LDS
// and each thread the coefficients and right-hand side of its nodes in
// registers.  A half-sweep is then five LDS accesses a node and a barrier.  The
// cycle is that of the passes (sweeps, residual, restriction, exact solve,
// prolongation, sweeps) and evaluates every node by the same expressions.
//
// What bounds it: latency, some 200 cycles of LDS reads, dependent arithmetic and
// a barrier a half-sweep.  A cycle takes 4.2 us at 33 x 16 x 33, where the passes,
// bound by the chain of operations of a chunk's rows and by the launches, take
// 13.6 us (merged) and 4 us (exact solve): 198 us the solve, 99 now.  With two
// column pairs a thread of 1024 the registers spill a little and the gain is
// less: 300 -> 216 us at 65 x 128 x 65, 279 -> 243 at 33 x 64 x 120; a third pair is
// not offered.
#include "direct_tile.h"
#include "stencil.h"

#include <algorithm>

namespace cp {

namespace {

struct PlaneArgs {
    LevelView v, vc;
    Transfer1D tr, tz;
    const double* lam;
    double* u;            // iterate: in (see start) and out
    const double* f;
    const double* ec;     // kStartPro: level 1's answer
    const double *V, *VT, *M;
    int nc;               // cosine planes
    double omega;
    int nu1, nu2, cycles, start;
    double* partial;      // the last cycle's squared residual, one sum a plane
    int partial_ld;
    const int* mask;
    int p0;
};

// The interior of the first cycle's iterate: u's own, zero, or interpolated from level 1.
enum PlaneStart { kStartFull = 0, kStartZero = 1, kStartPro = 2 };

constexpr int kMaxPairs = 2;  // column pairs of a thread

// One wavefront is the exact solve's below 17 nodes each way; 512 threads leave
// their registers room for every coefficient there.
int plane_threads(int g) { return g == 1 ? 512 : 1024; }

// The exact solve's tables are kept in LDS up to this G (48 KB there, twice as
// much beyond).
constexpr int kTablesG = 2;

size_t plane_lds(const LevelView& v, const LevelView& vc, int g) {
    size_t n = (size_t)2 * v.nr * v.nz + (size_t)vc.nr * vc.nz + (size_t)16 * g * (16 * g + 1) + 16;
    n += (size_t)5 * (v.nr + v.nz + 2) / 2 + (size_t)5 * (vc.nr + vc.nz + 2) / 2 + 2;  // transfer tables
    if (g <= kTablesG) n += (size_t)2 * g * 4 * g * 64 + (size_t)g * kSegRows * 16 * 4 * g;
    return n * sizeof(double);
}

// A transfer's tables in LDS.
struct Tables {
    double *pwl, *pwr, *rwm, *rwp;
    int *pidx, *cidx;
    __device__ __forceinline__ double* place(double* p, int nf, int nc) {
        pwl = p;
        pwr = pwl + nf;
        rwm = pwr + nf;
        rwp = rwm + nc;
        pidx = (int*)(rwp + nc);
        cidx = pidx + nf;
        return rwp + nc + (nf + nc + 1) / 2;
    }
    __device__ __forceinline__ void fill(const Transfer1D& t, int nf, int nc, int at, int step) {
        for (int q = at; q < nf; q += step) {
            pwl[q] = t.pwl[q];
            pwr[q] = t.pwr[q];
            pidx[q] = t.pidx[q];
        }
        for (int q = at; q < nc; q += step) {
            rwm[q] = t.rwm[q];
            rwp[q] = t.rwp[q];
            cidx[q] = t.cidx[q];
        }
    }
};

// G: interior nodes of level 1 up to 16 G each way; T threads; PM column pairs
// (one red and one black node each) of a thread.
template <int G, int T, int PM>
__global__ void __launch_bounds__(T) k_plane(PlaneArgs a) {
#pragma clang fp contract(off)
    constexpr int N = 16 * G, NSEG = 4 * G, KS = 4 * G, LD = N + 1;
    extern __shared__ double lds[];
    const LevelView &v = a.v, &vc = a.vc;
    const int plane = a.p0 + blockIdx.x;
    if (a.mask && a.mask[plane] == 0) return;  // whole workgroup, before any barrier
    const int nr = v.nr, nz = v.nz, nri = nr - 2, nzi = nz - 2;
    const int cnr = vc.nr, cnz = vc.nz, cnri = cnr - 2, cnzi = cnz - 2;
    double* const u = lds;             // [nz][nr]
    double* const r = u + nr * nz;     // [nz][nr], zero ring
    double* const e = r + nr * nz;     // [cnz][cnr], zero ring: coarse right-hand side, then answer
    double* const gs = e + cnr * cnz;  // [N][LD]
    double* const red = gs + N * LD;
    Tables tr, tz;
    double* next = tr.place(red + 16, nr, cnr);
    next = tz.place(next, nz, cnz);
    constexpr bool TAB = G <= kTablesG;
    constexpr int NV = G * KS * 64, NM = G * kSegRows * 16 * NSEG;
    double* const lv = next;           // V, VT and the plane's elimination factors
    const int t = threadIdx.x, wave = t >> 6, l = t & 63;
    double* const up = a.u + (long long)plane * v.pstride;
    const double* const fp = a.f + (long long)plane * v.pstride;
    const double lam = a.lam[plane];

    for (int q = t; q < nr * nz; q += T) {
        const int k = q / nr, i = q % nr;
        const bool in = i >= 1 && i <= nri && k >= 1 && k <= nzi;
        double x = 0.0;
        if (!in || a.start == kStartFull) x = up[(long long)k * v.pitch + i];
        if (in && a.start == kStartPro) {
            const double* c0 = a.ec + (long long)plane * vc.pstride + (long long)a.tz.pidx[k] * vc.pitch + a.tr.pidx[i];
            x = prolong_value(c0, vc.pitch, a.tr.pwl[i], a.tr.pwr[i], a.tz.pwl[k], a.tz.pwr[k]);
        }
        u[q] = x;
        r[q] = 0.0;
    }
    for (int q = t; q < cnr * cnz; q += T) e[q] = 0.0;
    tr.fill(a.tr, nr, cnr, t, T);
    tz.fill(a.tz, nz, cnz, t, T);
    const double* factors = a.M + (size_t)mode_of(plane, a.nc) * NM;
    const double *V = a.V, *VT = a.VT;
    if (TAB) {
        for (int q = t; q < NV; q += T) {
            lv[q] = V[q];
            lv[NV + q] = VT[q];
        }
        for (int q = t; q < NM; q += T) lv[2 * NV + q] = factors[q];
    }

    // this thread's nodes: pair m's red (colour 0, i + k even) and black one
    const int np = (nri + 1) / 2;
    int at[PM][2];       // position in the plane, 0 where there is none
    int row[PM];
    double f[PM][2], invd[PM][2];
    double rw[PM][2], re[PM][2], rb[PM][2], rm[PM][2], zc[PM], zs[PM], zn[PM];
#pragma unroll
    for (int m = 0; m < PM; ++m) {
        const int q = t + T * m, k = 1 + q / np, j = 2 * (q % np);
        row[m] = k;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int i = 1 + j + (((k & 1) ^ c) ^ 1);
            const bool on = k <= nzi && i <= nri;
            at[m][c] = on ? k * nr + i : 0;
            f[m][c] = on ? fp[(long long)k * v.pitch + i] : 0.0;
            const int ci = on ? i : 1, ck = on ? k : 1;
            rw[m][c] = v.rw[ci];
            re[m][c] = v.re[ci];
            rb[m][c] = v.rb[ci];
            rm[m][c] = v.rm[ci];
            invd[m][c] = coef_at(v, ci, ck, lam).invd;
            if (c == 0 || on) {
                zc[m] = v.zc[ck];
                zs[m] = v.zs[ck];
                zn[m] = v.zn[ck];
            }
        }
    }
    // a node's coefficients, formed where they are used: kept, they would not
    // fit the registers of 1024 threads
    auto coef = [&](int m, int c) {
        if (T == 1024) __asm__ volatile("" : "+v"(zc[m]));
        Coef k = make_coef_products(rw[m][c], re[m][c], rb[m][c], rm[m][c], zc[m], zs[m], zn[m], lam);
        k.invd = invd[m][c];
        return k;
    };
    // the exact solve: this lane's rows of an eigenvector
    const int chain = t / NSEG, seg = t % NSEG;
    const int mine = (chain / 16) * (kSegRows * 16 * NSEG) + t % (16 * NSEG);
    __syncthreads();

    auto sweeps = [&](int n) {
        for (int h = 0; h < n; ++h)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
#pragma unroll
                for (int m = 0; m < PM; ++m)
                    if (const int o = at[m][c])
                        u[o] = relax(u[o], f[m][c], u[o - 1], u[o + 1], u[o - nr], u[o + nr], coef(m, c), a.omega);
                __syncthreads();
            }
    };
    auto res = [&](int m, int c) {
        const int o = at[m][c];
        return residual(u[o], f[m][c], u[o - 1], u[o + 1], u[o - nr], u[o + nr], coef(m, c));
    };

    for (int cycle = 0; cycle < a.cycles; ++cycle) {
        // tables in global memory are loaded where they are used: kept from one
        // cycle to the next they would take the registers of the nodes
        if (!TAB) __asm__ volatile("" : "+s"(factors), "+s"(V), "+s"(VT));
        sweeps(a.nu1);
#pragma unroll
        for (int m = 0; m < PM; ++m)
#pragma unroll
            for (int c = 0; c < 2; ++c)
                if (at[m][c]) r[at[m][c]] = res(m, c);
        __syncthreads();
        for (int q = t; q < cnri * cnzi; q += T) {
            const int K = 1 + q / cnri, I = 1 + q % cnri;
            const double* rp = r + tz.cidx[K] * nr + tr.cidx[I];
            const double wm = tz.rwm[K], wp = tz.rwp[K];
            double col[3];
#pragma unroll
            for (int d = 0; d < 3; ++d) col[d] = restrict3(rp[d - 1 - nr], rp[d - 1], rp[d - 1 + nr], wm, wp);
            e[K * cnr + I] = restrict3(col[0], col[1], col[2], tr.rwm[I], tr.rwp[I]);
        }
        __syncthreads();
        // exact solve: transform, eliminations, inverse transform
        const int kr = l >> 4, cl = l & 15, grp = wave / G, col = 16 * (wave % G) + cl;
        const bool in = col < cnri;
        SegTables tb;
        if (t < 64 * G * G) tb.load(vc, (TAB ? lv + 2 * NV : factors) + mine, 16 * NSEG, seg);
        if (wave < G * G) {
            dbl4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const int k = 4 * s + kr;
                const double b = in && k < cnzi ? e[(k + 1) * cnr + 1 + col] : 0.0;
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64((TAB ? lv : V)[(grp * KS + s) * 64 + l], b, acc, 0, 0, 0);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) gs[(16 * grp + kr + 4 * q) * LD + col] = acc[q];
        }
        __syncthreads();
        if (t < 64 * G * G) {
            double g[kSegRows];
            double* mid = gs + chain * LD + seg * kSegRows;
#pragma unroll
            for (int q = 0; q < kSegRows; ++q) g[q] = mid[q];
            eliminate<NSEG>(tb, g, seg);
#pragma unroll
            for (int q = 0; q < kSegRows; ++q) mid[q] = g[q];
        }
        __syncthreads();
        if (wave < G * G) {
            dbl4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < KS; ++s)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64((TAB ? lv + NV : VT)[(grp * KS + s) * 64 + l],
                                                           gs[(4 * s + kr) * LD + col], acc, 0, 0, 0);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int k = 16 * grp + kr + 4 * q;
                if (in && k < cnzi) e[(k + 1) * cnr + 1 + col] = acc[q];
            }
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < PM; ++m)
#pragma unroll
            for (int c = 0; c < 2; ++c)
                if (const int o = at[m][c]) {
                    const int k = row[m], i = o - k * nr;
                    u[o] += prolong_value(e + tz.pidx[k] * cnr + tr.pidx[i], cnr, tr.pwl[i], tr.pwr[i],
                                          tz.pwl[k], tz.pwr[k]);
                }
        __syncthreads();
        sweeps(a.nu2);
    }

    // the answer, and the sum of its squared residuals in a fixed order
    double sum = 0.0;
#pragma unroll
    for (int m = 0; m < PM; ++m)
#pragma unroll
        for (int c = 0; c < 2; ++c)
            if (const int o = at[m][c]) {
                const double x = res(m, c);
                sum = fma(x, x, sum);
                up[(long long)row[m] * v.pitch + o - row[m] * nr] = u[o];
            }
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) sum += __shfl_xor(sum, w);
    if (l == 0) red[wave] = sum;
    __syncthreads();
    if (t == 0) {
        for (int w = 1; w < T / 64; ++w) sum += red[w];
        a.partial[(long long)plane * a.partial_ld] = sum;
    }
}

template <int G, int T, int PM>
hipError_t launch_plane_t(const PlaneArgs& a, int np, size_t lds, hipStream_t s) {
    hipError_t e = hipFuncSetAttribute((const void*)k_plane<G, T, PM>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    k_plane<G, T, PM><<<np, T, lds, s>>>(a);
    return hipGetLastError();
}

int plane_pairs(const cylpoisson_plan* p, int g) {
    const int pairs = (p->nz - 2) * ((p->nr - 1) / 2), T = plane_threads(g);
    return (pairs + T - 1) / T;
}

}  // namespace

// Planes up to which this is faster than the passes.  A plane's workgroup fills
// a compute unit, so that beyond 256 planes they take turns, which the passes do
// not: with one pair a thread it is faster all the same (17 x 1024 x 17: 2431 us
// the solve, 2493 by passes; 41 x 1024 x 41: 2574, 2648), with two only up to
// there (65 x 256 x 65: 303, 329; 65 x 320 x 65: 1052, 996).  With two pairs and the
// exact solve's tables read from L2 by every plane, up to 64 (72 x 64 x 56: 275,
// 283; 72 x 96 x 56: 313, 298; 72 x 128 x 56: 358, 307).  The solves beside this
// one in a batch do not enter: their number must not change a solve's norms.
int plane_most(int g, int pairs) { return pairs == 1 ? 1 << 30 : g <= kTablesG ? 256 : 64; }

// Merged cycles (without the option "timing", which takes the passes apart) on
// two levels, the second solved by one workgroup a plane, and
// a finest plane whose nodes fit a workgroup's registers and LDS.
bool plane_active(const cylpoisson_plan* p) {
    if (p->opt.timing || direct_level(p) != 1 || !fused_merge_ok(p)) return false;
    const DirectLevel& d = p->dir[p->opt.direct == 2 ? 1 : 0];
    const int g = direct_g(p->hl[1]), pairs = plane_pairs(p, g);
    return !d.big && pairs <= kMaxPairs && p->nt <= plane_most(g, pairs) && plane_lds(p->dl[0].v, p->dl[1].v, g) <= 150 * 1024;
}

hipError_t launch_plane(cylpoisson_plan* p, int cycles, bool zero_top, bool pro, double* partial, int partial_ld,
                        hipStream_t s) {
    const DirectLevel& d = p->dir[p->opt.direct == 2 ? 1 : 0];
    PlaneArgs a{};
    a.v = p->dl[0].v;
    a.vc = p->dl[1].v;
    a.tr = p->dl[0].tr;
    a.tz = p->dl[0].tz;
    a.lam = p->d_lam;
    a.u = p->dl[0].u;
    a.f = p->dl[0].f;
    a.ec = p->dl[1].u;
    a.V = d.V;
    a.VT = d.VT;
    a.M = d.M;
    a.nc = p->nt / 2 + 1;
    a.omega = p->opt.omega;
    a.nu1 = nu_pre(p, 0);
    a.nu2 = nu_post(p, 0);
    a.cycles = cycles;
    a.start = pro ? kStartPro : zero_top ? kStartZero : kStartFull;
    a.partial = partial;
    a.partial_ld = partial_ld;
    a.mask = p->mask_live ? p->d_mask : nullptr;
    const int g = direct_g(p->hl[1]), pm = plane_pairs(p, g);
    const size_t lds = plane_lds(a.v, a.vc, g);
    switch (g) {
        case 1: return pm == 1 ? launch_plane_t<1, 512, 1>(a, p->nt, lds, s) : launch_plane_t<1, 512, 2>(a, p->nt, lds, s);
        case 2: return pm == 1 ? launch_plane_t<2, 1024, 1>(a, p->nt, lds, s) : launch_plane_t<2, 1024, 2>(a, p->nt, lds, s);
        default: return pm == 1 ? launch_plane_t<4, 1024, 1>(a, p->nt, lds, s) : launch_plane_t<4, 1024, 2>(a, p->nt, lds, s);
    }
}

}  // namespace cp
