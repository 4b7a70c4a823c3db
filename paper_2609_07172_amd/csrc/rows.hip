// Single sweeps over a level's rows for gfx950: the plane norms, the refinement
// step of the mixed-precision solve, and the restriction of the finest
// right-hand side.
//
// One wavefront owns a strip of column pairs of one plane (62 pairs, one more
// lane on either side for the neighbours' values) and a chunk of rows, and
// marches along z: the rows below, at and above the evaluated one are the
// lane's registers, the horizontal neighbours come by cross-lane moves, and
// the next kAhead rows are in flight.  There is no LDS and no barrier.
//
// All are bound by HBM: each reads and writes every node's values once, except
// the two rows and columns that neighbouring chunks and strips share.
#include "fused_pass.h"

namespace cp {

namespace {

constexpr int kAhead = 4;         // rows in flight
constexpr int kRowWaves = 4096;   // wavefronts of a launch: four per SIMD (6144 and more lose 2% at 257 x 64 x 257)
constexpr int kStripPairs = 62;

struct RowShape {
    int chunk, nchunks, nstrips;  // rows per chunk; chunks and strips per plane
    int nb;                       // wavefronts per plane
    bool ok;                      // within the partial sums and the 32-bit offsets
    int bs;                       // of them side by side (a wavefront takes every bs-th strip)
};

// `most`: wavefronts per plane at most (one partial sum each); `wide`: rows too
// long for offsets within a chunk
RowShape row_shape(int rows, int nr, long long pitch, int nt, int most, bool wide = false) {
    RowShape s;
    const int pairs = (nr - 1) / 2 + 1;
    s.nstrips = pairs <= 64 ? 1 : (pairs - 2 + kStripPairs - 1) / kStripPairs;
    // side by side at most so many that a chunk's bytes fit the offsets below
    s.bs = std::min(s.nstrips, std::min(most, kMaxPartial) / 16);
    const int want = std::max(1, std::min(most, kRowWaves / std::max(1, nt)) / s.bs);
    s.chunk = std::max(kMinChunk, (rows + want - 1) / want);
    s.chunk = std::max(s.chunk, (rows + most / s.bs - 1) / (most / s.bs));
    // 32-bit byte offsets within a chunk
    if (!wide) s.chunk = (int)std::max(1LL, std::min<long long>(s.chunk, kMaxRange / (pitch * 8) - 2 * kAhead));
    s.nchunks = (rows + s.chunk - 1) / s.chunk;
    s.nb = s.nchunks * s.bs;
    s.ok = s.nb <= most && (wide || (s.chunk + 2LL) * pitch * 8 <= kMaxRange);
    return s;
}

struct RowArgs {
    LevelView v;
    RowShape sh;
    const double* lam;
    const double* u;
    const double* f;
    const float* e;
    double* out;
    float* r32;
    double* partial;   // [plane][kMaxPartial]: sums of r^2 ...
    double* partial2;  // ... and of b^2
};

// A wavefront's strip: its columns and their radial tables.
struct Strip {
    int p, chunk, strip0, za, zb;
    int c1;
    bool act[2], own;
    double rw[2], re[2], rb[2], rm[2];

    __device__ __forceinline__ void place(const RowShape& sh, const LevelView& v) {
        p = blockIdx.y;
        chunk = blockIdx.x / sh.bs;
        strip0 = blockIdx.x % sh.bs;
        za = 1 + chunk * sh.chunk;
        zb = min(v.nz - 1, za + sh.chunk);
    }
    __device__ __forceinline__ void columns(const RowShape& sh, const LevelView& v, int strip) {
        const int lane = threadIdx.x;
        c1 = 2 * (strip * kStripPairs + lane);
        own = (strip == 0 || lane > 0) && (strip == sh.nstrips - 1 || lane < 63);
        act[0] = c1 >= 1 && c1 <= v.nr - 2;
        act[1] = c1 + 1 <= v.nr - 2;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int i = act[c] ? c1 + c : 1;
            rw[c] = v.rw[i];
            re[c] = v.re[i];
            rb[c] = v.rb[i];
            rm[c] = v.rm[i];
        }
    }
};

// fixed-order sum over the wavefront
__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) x += __shfl_xor(x, w);
    return x;
}

// What a sweep evaluates.  kNormX: sums of f^2.  kNormR, kNormB, kNormBoth: sums of squares of the residual
// r = f - A u, of the right-hand side b (the residual of u's ring around a
// zero interior), or both.  kRefineZero, kRefineAsIs, kRefineAdd: sums of r^2
// and r rounded to FP32 for the iterate u's ring around a zero interior, u, or
// u + e (e zero on the ring), which the first and last also store into out.
enum RowMode { kNormX, kNormR, kNormB, kNormBoth, kRefineZero, kRefineAsIs, kRefineAdd };

// Measured: kRefineAdd at 257 x 64 x 257 moves 136 MB in 28.6 us and
// kRefineZero 85 MB in 18.7 us (34 and 29 as workgroups of a row's columns
// sharing rows through LDS, a barrier a row).  At 129 x 64 x 129, where launches
// count, kNormBoth and its sums take 9 + 3 us for what were a residual written
// and read again and three sums (37 us).
// WIDE (norms only): rows of hundreds of megabytes, whose loads take a buffer a
// row from the strip's first column on instead of one a chunk.
template <int MODE, bool WIDE>
__global__ void __launch_bounds__(64, 4) k_rows(RowArgs a) {
#pragma clang fp contract(off)
    static_assert(!WIDE || MODE <= kNormBoth, "the wide form stores nothing");
    constexpr bool RING = MODE == kNormB || MODE == kRefineZero;  // reads u's ring only
    constexpr bool U = MODE != kNormX;
    constexpr bool R = U && MODE != kNormB;
    constexpr bool B = MODE == kNormB || MODE == kNormBoth;
    constexpr bool REFINE = MODE == kRefineZero || MODE == kRefineAsIs || MODE == kRefineAdd;
    constexpr bool ADD = MODE == kRefineAdd;
    constexpr bool OUT = MODE == kRefineZero || ADD;
    const LevelView& v = a.v;
    Strip w;
    w.place(a.sh, v);
    const int za = w.za, zb = w.zb, s = za - 1;
    const double lam = U ? a.lam[w.p] : 0.0;
    const CTab zct = ctab(v.zc), zst = ctab(v.zs), znt = ctab(v.zn);
    // buffers from the row before the chunk on; rows are offsets from it
    const long long first = (long long)w.p * v.pstride + (long long)s * v.pitch;
    const long long left = (long long)(v.nz - s) * v.pitch;
    rsrc_t ru, re, ro, r3;
    if (U) ru = make_rsrc(a.u + first, left);
    const rsrc_t rf = make_rsrc(a.f + first, left);
    if (ADD) re = make_rsrc(a.e + first, left);
    if (OUT) ro = make_rsrc(a.out + first, left);
    if (REFINE) r3 = make_rsrc(a.r32 + first, left);
    const unsigned row8 = (unsigned)(v.pitch * 8), row4 = (unsigned)(v.pitch * 4);
    double acc = 0.0, accb = 0.0;
    for (int strip = w.strip0; strip < a.sh.nstrips; strip += a.sh.bs) {
        w.columns(a.sh, v, strip);
        const int c1 = w.c1;
        const bool a0 = w.act[0], a1 = w.act[1], any = a0 || a1;
        const int col0 = WIDE ? 2 * strip * kStripPairs : 0;
        const unsigned voff = c1 < v.nr ? (unsigned)(c1 - col0) * 8 : kOff;
        const unsigned vring = a0 && a1 ? kOff : voff;
        const unsigned vin = any ? voff : kOff, vin4 = any ? (unsigned)c1 * 4 : kOff;
        const unsigned vst = w.own ? vin : kOff, vst4 = w.own ? vin4 : kOff;
        // row xr, in the buffer `r` of the rows from `base` on
        auto load_row = [&](rsrc_t r, const double* base, unsigned off, int xr) {
            if constexpr (WIDE)
                return load2<double>(make_rsrc(base + (long long)(xr - s) * v.pitch + col0,
                                               (long long)(v.nz - xr) * v.pitch - col0), off, 0);
            else
                return load2<double>(r, off, (unsigned)(xr - s) * row8);
        };
        auto load_u = [&](int x) -> Pair<double> {
            if (!U) return {0.0, 0.0};
            const int xr = min(x, zb);
            return load_row(ru, a.u + first, RING && xr >= 1 && xr <= v.nz - 2 ? vring : voff, xr);
        };
        auto load_e = [&](int x) -> Pair<float> {
            const int xr = min(x, zb);
            return load2<float>(re, xr >= 1 && xr <= v.nz - 2 ? vin4 : kOff, (unsigned)(xr - s) * row4);
        };
        auto load_f = [&](int x) { return load_row(rf, a.f + first, vin, min(x, zb)); };
        // the iterate of a loaded row
        auto value = [&](int x, const Pair<double>& l, const Pair<float>& d, double (&o)[2]) {
            const bool in = x >= 1 && x <= v.nz - 2;
            o[0] = l.a;
            o[1] = l.b;
            if (RING) {
                if (in && a0) o[0] = 0.0;
                if (in && a1) o[1] = 0.0;
            }
            if (ADD) {
                if (in && a0) o[0] = l.a + (double)d.a;
                if (in && a1) o[1] = l.b + (double)d.b;
            }
        };
        Pair<double> pu[kAhead], pf[kAhead];
        Pair<float> pe[kAhead];
        double lo[2], mid[2], hi[2];
        {
            const Pair<double> l0 = load_u(s), l1 = load_u(za);
            Pair<float> e0{}, e1{};
            if (ADD) {
                e0 = load_e(s);
                e1 = load_e(za);
            }
#pragma unroll
            for (int j = 0; j < kAhead; ++j) {
                pu[j] = load_u(za + 1 + j);
                if (ADD) pe[j] = load_e(za + 1 + j);
                pf[j] = load_f(za + j);
            }
            value(s, l0, e0, lo);
            value(za, l1, e1, mid);
        }
        for (int x0 = za; x0 < zb; x0 += kAhead) {
#pragma unroll
            for (int j = 0; j < kAhead; ++j) {
                const int x = x0 + j;
                value(x + 1, pu[j], pe[j], hi);
                const Pair<double> f = pf[j];
                pu[j] = load_u(x + 1 + kAhead);
                if (ADD) pe[j] = load_e(x + 1 + kAhead);
                pf[j] = load_f(x + kAhead);
                if (x < zb) {
                    const double zc = zct[x], zs = zst[x], zn = znt[x];
                    const Coef k0 = make_coef_products(w.rw[0], w.re[0], w.rb[0], w.rm[0], zc, zs, zn, lam);
                    const Coef k1 = make_coef_products(w.rw[1], w.re[1], w.rb[1], w.rm[1], zc, zs, zn, lam);
                    const double west = from_lane<true>(mid[1]), east = from_lane<false>(mid[0]);
                    const unsigned so = (unsigned)(x - s) * row8;
                    if (R) {
                        const double r0 = residual(mid[0], f.a, west, mid[1], lo[0], hi[0], k0);
                        const double r1 = residual(mid[1], f.b, mid[0], east, lo[1], hi[1], k1);
                        const double d0 = a0 ? r0 : 0.0, d1 = a1 ? r1 : 0.0;
                        if (REFINE) store2<float>(r3, vst4, (unsigned)(x - s) * row4, (float)d0, (float)d1);
                        if (REFINE && OUT) store2<double>(ro, vst, so, mid[0], mid[1]);
                        if (w.own) {
                            acc = fma(d0, d0, acc);
                            acc = fma(d1, d1, acc);
                        }
                    }
                    if (MODE == kNormX && w.own) {
                        if (a0) acc = fma(f.a, f.a, acc);
                        if (a1) acc = fma(f.b, f.b, acc);
                    }
                    if (B) {
                        // the interior taken as zero
                        const double m0 = a0 ? 0.0 : mid[0], m1 = a1 ? 0.0 : mid[1];
                        const double mw = from_lane<true>(m1), me = from_lane<false>(m0);
                        const bool lr = x == 1, hr = x == v.nz - 2;
                        const double r0 = residual(0.0, f.a, mw, m1, lr ? lo[0] : 0.0, hr ? hi[0] : 0.0, k0);
                        const double r1 = residual(0.0, f.b, m0, me, lr ? lo[1] : 0.0, hr ? hi[1] : 0.0, k1);
                        if (w.own && a0) accb = fma(r0, r0, accb);
                        if (w.own && a1) accb = fma(r1, r1, accb);
                    }
                }
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    lo[c] = mid[c];
                    mid[c] = hi[c];
                }
            }
        }
    }
    if (R || MODE == kNormX) {
        acc = wave_sum(acc);
        if (threadIdx.x == 0) a.partial[(long long)w.p * kMaxPartial + blockIdx.x] = acc;
    }
    if (B) {
        accb = wave_sum(accb);
        if (threadIdx.x == 0) a.partial2[(long long)w.p * kMaxPartial + blockIdx.x] = accb;
    }
}

// ---- the finest right-hand side's restriction and norms ----
struct RestrictArgs {
    LevelView v, vc;
    Transfer1D tr, tz;
    RowShape sh;  // chunks of coarse rows
    const double* lam;
    const double* u;
    const double* f;
    double* fc;
    double* partial;
    int rc;  // coarsened in r
};

// f_c = P^T b for the residual b of the iterate that is u's ring and zero
// inside, and the sums of b^2 over the fine interior, in one pass over f.
// Only plane 0 has a non-zero ring (theta-invariant face values), so on every
// other plane b = f exactly and u is not read.  A coarse node lies on fine row
// and column 2K, 2I (ZC, rc; else K, I), and is the vertical three-point sum of
// each column, then the horizontal one, as in every other restriction.  A fine
// row counts for the chunk of the coarse row on or above it.
// 8 B a fine node read and 2 B written: 67 us at 400 x 128 x 512 (262 MB; 94 us
// as a workgroup a block of coarse columns with rows in LDS and a barrier a row,
// and two more launches for plane 0's nodes next to a face).
template <bool ZC>
__global__ void __launch_bounds__(64, 4) k_restrict_rhs(RestrictArgs a) {
#pragma clang fp contract(off)
    constexpr int S = ZC ? 2 : 1;  // fine rows per coarse row
    constexpr int A = kAhead / S;  // coarse rows in flight
    const LevelView& v = a.v;
    Strip w;
    w.place(a.sh, a.vc);
    const int Ka = w.za, Kb = w.zb, ke = v.nz - 2;
    const int s = S * Ka - (S - 1);  // the chunk's first fine row
    const bool ringed = w.p == 0;
    const double lam = a.lam[w.p];
    const CTab zct = ctab(v.zc), zst = ctab(v.zs), znt = ctab(v.zn);
    const CTab rwm = ctab(a.tz.rwm), rwp = ctab(a.tz.rwp);
    const long long first = (long long)w.p * v.pstride + (long long)s * v.pitch;
    const long long left = (long long)(v.nz - s) * v.pitch;
    const rsrc_t rf = make_rsrc(a.f + first, left);
    const rsrc_t ru = make_rsrc(a.u + first, left);
    const rsrc_t rc = make_rsrc(a.fc + (long long)w.p * a.vc.pstride + (long long)Ka * a.vc.pitch,
                                (long long)(a.vc.nz - Ka) * a.vc.pitch);
    const unsigned row8 = (unsigned)(v.pitch * 8), crow8 = (unsigned)(a.vc.pitch * 8);
    const int last = min(S * Kb - 1, ke);                         // last fine row read
    const int counted = Kb == a.vc.nz - 1 ? ke : S * Kb - S;      // last fine row counted
    double acc = 0.0;
    for (int strip = w.strip0; strip < a.sh.nstrips; strip += a.sh.bs) {
        w.columns(a.sh, v, strip);
        const int c1 = w.c1, e0 = a.rc ? c1 / 2 : c1;
        const bool a0 = w.act[0], a1 = w.act[1], any = a0 || a1;
        const unsigned vin = any ? (unsigned)c1 * 8 : kOff;
        const unsigned vring = ringed && any && !(a0 && a1) ? vin : ringed && c1 == v.nr - 1 ? (unsigned)c1 * 8 : kOff;
        const bool in = w.own && e0 >= 1 && e0 <= a.vc.nr - 2;
        const unsigned vfc = (a.rc ? in : w.own && any) ? (unsigned)e0 * 8 : kOff;
        const double wrm = a.rc && in ? a.tr.rwm[e0] : 0.0, wrp = a.rc && in ? a.tr.rwp[e0] : 0.0;
        auto load = [&](rsrc_t r, unsigned off, int k) { return load2<double>(r, off, (unsigned)(min(k, last) - s) * row8); };
        // b of a loaded row
        auto rhs = [&](int k, const Pair<double>& l, const Pair<double>& ring, double (&o)[2]) {
            o[0] = a0 ? l.a : 0.0;
            o[1] = a1 ? l.b : 0.0;
            if (ringed) {
                const double m0 = a0 ? 0.0 : ring.a, m1 = a1 ? 0.0 : ring.b;
                Pair<double> lo{0.0, 0.0}, hi{0.0, 0.0};
                const double* plane = a.u;  // plane 0
                if (k == 1 && any) lo = {plane[c1], plane[c1 + 1]};
                if (k == ke && any) {
                    const double* q = plane + (long long)(ke + 1) * v.pitch + c1;
                    hi = {q[0], q[1]};
                }
                const double west = from_lane<true>(m1), east = from_lane<false>(m0);
                const double zc = zct[k], zs = zst[k], zn = znt[k];
                const Coef k0 = make_coef_products(w.rw[0], w.re[0], w.rb[0], w.rm[0], zc, zs, zn, lam);
                const Coef k1 = make_coef_products(w.rw[1], w.re[1], w.rb[1], w.rm[1], zc, zs, zn, lam);
                o[0] = a0 ? residual(0.0, o[0], west, m1, lo.a, hi.a, k0) : 0.0;
                o[1] = a1 ? residual(0.0, o[1], m0, east, lo.b, hi.b, k1) : 0.0;
            }
            if (w.own && k <= counted) {
                acc = fma(o[0], o[0], acc);
                acc = fma(o[1], o[1], acc);
            }
        };
        Pair<double> pf[A][S], pr[A][S];
        double below[2] = {0.0, 0.0};
        if (ZC) rhs(s, load(rf, vin, s), load(ru, vring, s), below);
        const int k0 = S * Ka;
#pragma unroll
        for (int j = 0; j < A; ++j)
#pragma unroll
            for (int i = 0; i < S; ++i) {
                pf[j][i] = load(rf, vin, k0 + S * j + i);
                pr[j][i] = load(ru, vring, k0 + S * j + i);
            }
        for (int K0 = Ka; K0 < Kb; K0 += A) {
#pragma unroll
            for (int j = 0; j < A; ++j) {
                const int K = K0 + j, k = S * K;
                Pair<double> l[S], g[S];
#pragma unroll
                for (int i = 0; i < S; ++i) {
                    l[i] = pf[j][i];
                    g[i] = pr[j][i];
                    pf[j][i] = load(rf, vin, k + S * A + i);
                    pr[j][i] = load(ru, vring, k + S * A + i);
                }
                if (K >= Kb) continue;
                double on[2], above[2] = {0.0, 0.0}, x[2];
                rhs(k, l[0], g[0], on);
                x[0] = on[0];
                x[1] = on[1];
                if (ZC) {
                    if (k + 1 <= ke) rhs(k + 1, l[1], g[1], above);
                    const double wm = rwm[K], wp = rwp[K];
                    x[0] = restrict3(below[0], on[0], above[0], wm, wp);
                    x[1] = restrict3(below[1], on[1], above[1], wm, wp);
                    below[0] = above[0];
                    below[1] = above[1];
                }
                const unsigned so = (unsigned)(K - Ka) * crow8;
                if (a.rc)
                    store1<double>(rc, vfc, so, restrict3(from_lane<true>(x[1]), x[0], x[1], wrm, wrp));
                else
                    store2<double>(rc, vfc, so, x[0], x[1]);
            }
        }
    }
    acc = wave_sum(acc);
    if (threadIdx.x == 0) a.partial[(long long)w.p * kMaxPartial + blockIdx.x] = acc;
}

// Sums of a plane's partials, one wavefront per plane (one thread's serial sum
// took 7 us of latency where this takes 3): out[p] of the first nb
// and, with out2, out2[p] of the nb from `second` on.
__global__ void __launch_bounds__(64) k_norm_final(const double* __restrict__ partial, int nb, int second,
                                                   double* __restrict__ out, double* __restrict__ out2) {
    const int p = blockIdx.x;
    const double* q = partial + (long long)p * kMaxPartial;
    double a = 0.0, b = 0.0;
    for (int k = threadIdx.x; k < nb; k += 64) {
        a += q[k];
        if (out2) b += q[second + k];
    }
    a = wave_sum(a);
    if (out2) b = wave_sum(b);
    if (threadIdx.x == 0) {
        out[p] = a;
        if (out2) out2[p] = b;
    }
}

template <int MODE>
hipError_t launch_rows(RowArgs& a, int nt, int most, hipStream_t s) {
    if constexpr (MODE <= kNormBoth)
        if (!a.sh.ok) {
            a.sh = row_shape(a.v.nz - 2, a.v.nr, a.v.pitch, nt, most, true);
            k_rows<MODE, true><<<dim3(a.sh.nb, nt), 64, 0, s>>>(a);
            return hipGetLastError();
        }
    if (!a.sh.ok) return hipErrorInvalidValue;  // (the refinement: fused levels only, whose rows are short)
    k_rows<MODE, false><<<dim3(a.sh.nb, nt), 64, 0, s>>>(a);
    return hipGetLastError();
}

RowArgs row_args(const DeviceLevel& L, int nt, const double* lam, int most) {
    RowArgs a{};
    a.v = L.v;
    a.sh = row_shape(L.v.nz - 2, L.v.nr, L.v.pitch, nt, most);
    a.lam = lam;
    return a;
}

}  // namespace

hipError_t launch_norm_final(const double* partial, int nb, int nt, double* out, hipStream_t s) {
    k_norm_final<<<nt, 64, 0, s>>>(partial, nb, 0, out, nullptr);
    return hipGetLastError();
}

hipError_t launch_plane_norms(const DeviceLevel& L, int nt, const double* x, double* partial,
                              double* norms_out, hipStream_t s) {
    RowArgs a = row_args(L, nt, nullptr, kMaxPartial);
    a.f = x;
    a.partial = partial;
    const hipError_t e = launch_rows<kNormX>(a, nt, kMaxPartial, s);
    return e != hipSuccess ? e : launch_norm_final(partial, a.sh.nb, nt, norms_out, s);
}

hipError_t launch_norms(const DeviceLevel& L, int nt, const double* lam, const double* u, const double* f,
                        double* partial, double* r_norms, double* b_norms, hipStream_t s) {
    const bool both = r_norms && b_norms;
    const int most = both ? kMaxPartial / 2 : kMaxPartial;
    RowArgs a = row_args(L, nt, lam, most);
    a.u = u;
    a.f = f;
    a.partial = partial;
    a.partial2 = both ? partial + kMaxPartial / 2 : partial;
    const hipError_t e = both      ? launch_rows<kNormBoth>(a, nt, most, s)
                         : r_norms ? launch_rows<kNormR>(a, nt, most, s)
                                   : launch_rows<kNormB>(a, nt, most, s);
    if (e != hipSuccess) return e;
    k_norm_final<<<nt, 64, 0, s>>>(partial, a.sh.nb, kMaxPartial / 2, r_norms ? r_norms : b_norms,
                                   both ? b_norms : nullptr);
    return hipGetLastError();
}

hipError_t launch_restrict_rhs_norms(const DeviceLevel& F, const DeviceLevel& C, int nt, const double* lam,
                                     const double* u, const double* f, double* fc, double* partial,
                                     double* norms_out, hipStream_t s) {
    RestrictArgs a{};
    a.v = F.v;
    a.vc = C.v;
    a.tr = F.tr;
    a.tz = F.tz;
    const bool zc = C.v.nz < F.v.nz;
    a.sh = row_shape(C.v.nz - 2, F.v.nr, (zc ? 2LL : 1LL) * F.v.pitch, nt, kMaxPartial);
    a.lam = lam;
    a.u = u;
    a.f = f;
    a.fc = fc;
    a.partial = partial;
    a.rc = C.v.nr < F.v.nr;
    if (!a.sh.ok) return hipErrorInvalidValue;
    const dim3 grid(a.sh.nb, nt);
    if (zc)
        k_restrict_rhs<true><<<grid, 64, 0, s>>>(a);
    else
        k_restrict_rhs<false><<<grid, 64, 0, s>>>(a);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : launch_norm_final(partial, a.sh.nb, nt, norms_out, s);
}

hipError_t launch_refine(const DeviceLevel& L, int nt, const double* lam, const double* uin,
                         double* uout, const float* e, const double* f, float* r32, double* partial,
                         double* norms_out, hipStream_t s) {
    RowArgs a = row_args(L, nt, lam, kMaxPartial);
    a.u = uin;
    a.f = f;
    a.e = e;
    a.out = uout;
    a.r32 = r32;
    a.partial = partial;
    if (e && uin == uout) return hipErrorInvalidValue;
    const hipError_t err = e      ? launch_rows<kRefineAdd>(a, nt, kMaxPartial, s)
                           : uout ? launch_rows<kRefineZero>(a, nt, kMaxPartial, s)
                                  : launch_rows<kRefineAsIs>(a, nt, kMaxPartial, s);
    return err != hipSuccess ? err : launch_norm_final(partial, a.sh.nb, nt, norms_out, s);
}

}  // namespace cp
