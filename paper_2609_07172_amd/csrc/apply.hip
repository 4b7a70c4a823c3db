// The discrete 3-D operator for gfx950: the seven-point cell balance of App. A
// with the azimuthal three-point term, on the node array itself.  The modes'
// shifts 4 / dtheta^2 sin^2(m dtheta / 2) are the eigenvalues of that term, so
// this is the operator that the mode path solves, without the two transforms.
//
// One wavefront owns a strip of column pairs (62, one more lane on either side
// for the neighbours' values), kRows axial rows and a run of planes, and marches
// along theta: the plane before, at and after the evaluated one are the lane's
// registers, and the one after that is in flight.  Horizontal neighbours come by
// cross-lane moves, the rows above and below the block are loaded with it.
// Consecutive blocks of rows run on one XCD, whose L2 serves the shared rows.
//
// Bound by HBM: 8 B a node read and written, besides two planes a run.
// 257 x 128 x 257 takes 29 us for its 135 MB (4.7 TB/s; the transforms and the
// planes' operator between them moved three times that in 105 us).
#include "fused_pass.h"

namespace cp {

namespace {

constexpr int kRows = 4;          // axial rows of a wavefront
constexpr int kStripPairs = 62;
constexpr int kApplyWaves = 2048; // about this many wavefronts in all ...
constexpr int kMinRun = 8;        // ... of at least this many planes (two more are read)

struct ApplyArgs {
    LevelView v;
    const double* u;
    const double* inv_s;
    double* out;
    double dt2;                    // 1 / dtheta^2
    int nt, run, nruns, nblocks, nstrips;
    int units;                     // runs x blocks of rows x strips
};

// WIDE: rows of hundreds of megabytes, too long for 32-bit offsets within a block
// of them: a buffer a row from the strip's first column on instead of one a block.
template <bool WIDE>
__global__ void __launch_bounds__(64, 2) k_apply(ApplyArgs a) {
#pragma clang fp contract(off)
    const LevelView& v = a.v;
    const int per = (a.units + 7) / 8;
    const int unit = ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);
    if (((int)blockIdx.x >> 3) >= per || unit >= a.units) return;
    const int strip = unit % a.nstrips, block = unit / a.nstrips % a.nblocks, run = unit / (a.nstrips * a.nblocks);
    const int lane = threadIdx.x, c1 = 2 * (strip * kStripPairs + lane);
    const bool own = (strip == 0 || lane > 0) && (strip == a.nstrips - 1 || lane < 63);
    const bool act[2] = {c1 >= 1 && c1 <= v.nr - 2, c1 + 1 <= v.nr - 2};
    const int z0 = 1 + block * kRows, s = z0 - 1;
    const int ja = run * a.run, jb = min(a.nt, ja + a.run);
    const unsigned row8 = (unsigned)(v.pitch * 8);
    const long long left = (long long)(v.nz - s) * v.pitch;
    const int col0 = WIDE ? 2 * strip * kStripPairs : 0;
    const unsigned voff = c1 < v.nr ? (unsigned)(c1 - col0) * 8 : kOff;
    // the buffer of an array's rows from row s on, of which `base` is the first; row y in it
    auto rows = [&](const double* base) { return make_rsrc(base, left); };
    auto row = [&](rsrc_t r, const double* base, int y) {
        if constexpr (WIDE)
            return make_rsrc(base + (long long)(y - s) * v.pitch + col0, (long long)(v.nz - y) * v.pitch - col0);
        else
            return r;
    };
    auto offset = [&](int y) { return WIDE ? 0u : (unsigned)(y - s) * row8; };
    const unsigned vst = own && c1 + 1 < v.nr ? voff : kOff;     // whole pairs
    const unsigned vlast = own && c1 == v.nr - 1 ? voff : kOff;  // the last column of an odd count
    double rw[2], re[2], rb[2], rm[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int i = act[c] ? c1 + c : 1;
        rw[c] = v.rw[i];
        re[c] = v.re[i];
        rb[c] = v.rb[i];
        rm[c] = v.rm[i];
    }
    const CTab zct = ctab(v.zc), zst = ctab(v.zs), znt = ctab(v.zn);
    double zc[kRows], zs[kRows], zn[kRows];
    double is[kRows][2];  // 1 / s; zero on the ring
    {
        const double* base = a.inv_s + (long long)s * v.pitch;
        const rsrc_t ri = rows(base);
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
            const int y = min(z0 + k, v.nz - 1);
            zc[k] = zct[y];
            zs[k] = zst[y];
            zn[k] = znt[y];
            const Pair<double> p = load2<double>(row(ri, base, y), voff, offset(y));
            is[k][0] = act[0] && z0 + k <= v.nz - 2 ? p.a : 0.0;
            is[k][1] = act[1] && z0 + k <= v.nz - 2 ? p.b : 0.0;
        }
    }
    // rows z0 - 1 .. z0 + kRows of plane j (rows past the last repeat it)
    auto load = [&](int j, Pair<double> (&o)[kRows + 2]) {
        const int q = j < 0 ? j + a.nt : j >= a.nt ? j - a.nt : j;
        const double* base = a.u + (long long)q * v.pstride + (long long)s * v.pitch;
        const rsrc_t r = rows(base);
#pragma unroll
        for (int k = 0; k < kRows + 2; ++k) {
            const int y = min(z0 - 1 + k, v.nz - 1);
            o[k] = load2<double>(row(r, base, y), voff, offset(y));
        }
    };
    Pair<double> before[kRows + 2], at[kRows + 2], after[kRows + 2], next[kRows + 2];
    load(ja - 1, before);
    load(ja, at);
    load(ja + 1, after);
    for (int j = ja; j < jb; ++j) {
        if (j + 1 < jb) load(j + 2, next);
        const double* base = a.out + (long long)j * v.pstride + (long long)s * v.pitch;
        const rsrc_t ro = rows(base);
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
            const Pair<double> m = at[k + 1];
            const double west = from_lane<true>(m.b), east = from_lane<false>(m.a);
            const double t0 = (m.a - before[k + 1].a) + (m.a - after[k + 1].a);
            const double t1 = (m.b - before[k + 1].b) + (m.b - after[k + 1].b);
            const Coef k0 = make_coef_products(rw[0], re[0], rb[0], rm[0], zc[k], zs[k], zn[k], 0.0);
            const Coef k1 = make_coef_products(rw[1], re[1], rb[1], rm[1], zc[k], zs[k], zn[k], 0.0);
            const double o0 = fma((rm[0] * zc[k]) * a.dt2, t0, apply_row(m.a, west, m.b, at[k].a, at[k + 2].a, k0));
            const double o1 = fma((rm[1] * zc[k]) * a.dt2, t1, apply_row(m.b, m.a, east, at[k].b, at[k + 2].b, k1));
            if (z0 + k <= v.nz - 2) {
                const rsrc_t r = row(ro, base, z0 + k);
                const unsigned so = offset(z0 + k);
                store2<double>(r, vst, so, act[0] ? o0 * is[k][0] : 0.0, act[1] ? o1 * is[k][1] : 0.0);
                store1<double>(r, vlast, so, 0.0);
            }
        }
        if (z0 == 1) {
            const rsrc_t r = row(ro, base, 0);
            store2<double>(r, vst, 0, 0.0, 0.0);
            store1<double>(r, vlast, 0, 0.0);
        }
        if (z0 + kRows >= v.nz - 1) {
            const rsrc_t r = row(ro, base, v.nz - 1);
            const unsigned so = offset(v.nz - 1);
            store2<double>(r, vst, so, 0.0, 0.0);
            store1<double>(r, vlast, so, 0.0);
        }
#pragma unroll
        for (int k = 0; k < kRows + 2; ++k) {
            before[k] = at[k];
            at[k] = after[k];
            after[k] = next[k];
        }
    }
}

}  // namespace

hipError_t launch_apply(const DeviceLevel& L, int nt, double dtheta, const double* u, const double* inv_s, double* out,
                        hipStream_t s) {
    ApplyArgs a{};
    a.v = L.v;
    a.u = u;
    a.inv_s = inv_s;
    a.out = out;
    a.dt2 = 1.0 / (dtheta * dtheta);
    a.nt = nt;
    const int pairs = (L.v.nr - 1) / 2 + 1;
    a.nstrips = pairs <= 64 ? 1 : (pairs - 2 + kStripPairs - 1) / kStripPairs;
    a.nblocks = (L.v.nz - 2 + kRows - 1) / kRows;
    const long long tiles = (long long)a.nstrips * a.nblocks;
    const int want = (int)std::max(1LL, std::min<long long>(nt, kApplyWaves / tiles));
    a.run = std::min(nt, std::max(kMinRun, (nt + want - 1) / want));
    a.nruns = (nt + a.run - 1) / a.run;
    a.units = (int)(tiles * a.nruns);
    const int blocks = 8 * ((a.units + 7) / 8);
    if ((kRows + 2LL) * L.v.pitch * 8 <= kMaxRange)  // 32-bit byte offsets within a block of rows
        k_apply<false><<<blocks, 64, 0, s>>>(a);
    else
        k_apply<true><<<blocks, 64, 0, s>>>(a);
    return hipGetLastError();
}

}  // namespace cp
