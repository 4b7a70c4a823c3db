// Fused streaming multigrid passes for gfx950.
//
// One wavefront owns a strip of radial columns of one plane and a chunk of
// axial rows: lane j holds the columns 2t and 2t + 1, t = t0 + j, of the last
// few rows in registers, and the wavefront marches along z.  At step x it
// consumes row x and, in the same step, runs every red-black half-sweep of
// the pass on the rows behind it (half-sweep h on row x - 1 - h), then the
// residual and the grid transfer, so all sweeps of a pass stream u and f
// through registers once.  Vertical neighbours are the lane's own registers;
// the horizontal neighbour from another lane comes through a cross-lane move,
// so there is no LDS row, no barrier and no coupling between wavefronts: each
// waits for its own loads only.  A half-sweep reads only values of earlier
// half-sweeps, in the order of the global red-black schedule (the arithmetic
// of every node is that of kernels.hip).
//
// Down pass (level l -> l+1): nu1 sweeps, residual, restriction f_{l+1} = P^T r.
// Up pass (level l): u += P e_{l+1}, nu2 sweeps, optional residual norm.
// Merged pass (finest level): the up pass of one cycle and the down pass of
// the next back to back.
//
// Strips and chunks overlap and recompute the overlap from the input iterate
// (outputs go to another buffer).  With H = 2 nu half-sweeps, a value next to
// a strip's open edge is wrong after one half-sweep and the error moves one
// column per half-sweep, so of a strip's 64 lanes nu + 1 on each open side
// are recomputed; a chunk [za, zb) starts H + 2 rows early and reads H + 1
// rows beyond.
//
// What bounds a pass.  At 400 x 128 x 512 (four strips a plane, two wavefronts
// per SIMD) the passes stream at 3.6 - 4.3 TB/s where a large copy reaches
// 5.1: the merged pass takes 182 us for its 727 MB (292 us as one workgroup per
// plane and chunk with rows exchanged through LDS, a barrier and several LDS
// round trips per row, at one wavefront per SIMD), the up pass 159 us (160),
// the first down pass 144 us (169).  On small grids the chain of dependent
// operations of one step times the rows of a chunk bounds it: 21 us merged at
// 129 x 64 x 129 (85 us: 64-row chunks, and unrolled code that was fetched once per
// step).
//
// Coarsening keeps every even node (and the last one), in z always 2:1 or not
// at all (ZC), in r likewise (args.rc), so a fine column or row 2I lies on the
// coarse one I and 2I + 1 between I and I + 1: the passes form these indices
// and read only the weights from the transfer tables.
//
// The pass is generic in the value type T of the iterate, right-hand side and
// transfers: double on the FP64 path, float in the inner V-cycles of the
// mixed-precision solve.  Coefficients are formed in double from the level's
// tables and rounded once to T.
#pragma once

#include <algorithm>
#include <type_traits>

#include "cp_internal.h"
#include "stencil.h"

namespace cp {

template <typename T>
struct PassArgs {
    LevelView v;   // this level
    LevelView vc;  // next coarser level
    Transfer1D tr, tz;
    const T* u_in;
    const T* f;
    T* u_out;
    T* fc;               // down: coarse right-hand side
    const T* ec;         // up: coarse correction
    const double* lam;
    const double* zrow;  // {zc, zs, zn, 0} of every row, kRowPad rows of zeros before row 0 and after the last
    int rc;              // the coarse level is coarsened in r
    int reg_lo, reg_hi;  // rows reg_lo <= y < reg_hi share the axial coefficients (zc0, zs0, zn0)
    double* partial;     // up: per (plane, chunk, strip) sum of squared residuals, or nullptr
    int partial_ld;      // stride between planes in `partial`
    double omega, zc0, zs0, zn0;
    int chunk, nchunks, nstrips;  // rows per chunk, chunks and strips per plane
    int p0;              // first plane of this launch
    const int* mask;     // per plane: 0 = frozen (its wavefronts return at once), or nullptr
    int xcd_major;       // the wavefronts of a plane run on one XCD
};

// Passes by kind: the input iterate and what the pass does.
enum PassKind { kDownZero = 0, kDownRing = 1, kDownFull = 2, kDownPro = 3, kUp = 4, kMerge = 5 };

// Where a level's coefficients come from.  kOneBand: every interior row is in
// the regular band, whose coefficients stay in registers.  kSomeRows: the few
// rows outside the band (next to a face) form theirs from the tables where
// they are used, in steps of their own.  kRowTables: every row's coefficients
// come from its tables in all steps; each row's two inverse diagonals are
// formed once, when the row is consumed, and stay in LDS (a ring of rows, 16 KB
// a wavefront: each lane reads its own, and as registers they and their moves
// would leave one wavefront a SIMD), and the row tables are four doubles a row
// with padding on both sides, so that a step reads them in a few scalar loads
// without bounds.
//
// Steps in the band cost less, a row outside it about a microsecond: with two
// rows outside (400 x 128 x 512, cells) the finest up pass takes 150 us as
// kSomeRows and 172 us as kRowTables, at 201 x 128 x 257 the down and up pass
// with one 36 and 40 us against 47 and 43, but with 54 rows outside 109 and 80
// against 51 and 46.  A merged pass of kSomeRows does not fit two wavefronts a
// SIMD and is slower on every mesh (129 x 64 x 129: 547 us the solve, 472 as
// kRowTables).
// Stretched 400 x 128 x 512: merged pass 205 us (inverse diagonals in
// registers and the tables row by row: 358, one wavefront a SIMD), level 1 down
// and up 47 and 43 us (57 and 42).
enum CoefMode { kOneBand = 0, kSomeRows = 1, kRowTables = 2 };

struct Shape {
    int chunk, nchunks, nstrips, per_plane;  // per_plane: wavefronts (= blocks) per plane
    bool zc;   // the next level is coarsened in z
    int coef;  // CoefMode
};

// Passes with a sweep count other than the default's two (four merged); fused_nu.hip.
hipError_t launch_other(int kind, int nu, bool fine, const Shape& sh, const PassArgs<double>& a, int np, hipStream_t s);

namespace {

// Lanes of a strip that no neighbouring strip owns, for nu sweeps.
constexpr int strip_step(int nu) { return 62 - 2 * nu; }

constexpr int kPassWaves = 2048;  // wavefronts of an automatic launch shape at two per SIMD
constexpr int kMinChunk = 4;      // rows per chunk at least
constexpr int kShortChunk = 20;   // rows of a merged chunk up to which one wavefront a SIMD is enough
constexpr int kFewRows = 4;       // rows outside the band that kSomeRows serves: two next to each face

// ---- buffer access: a scalar base and range, 32-bit lane and row offsets ----
// Accesses beyond the range read zero and write nothing, so a lane or row is
// switched off through its offset and every load and store is issued.
using rsrc_t = __amdgpu_buffer_rsrc_t;
constexpr unsigned kOff = 0x80000000u;       // beyond every range
constexpr long long kMaxRange = 0x7fff0000;  // bytes

template <typename T>
__device__ __forceinline__ rsrc_t make_rsrc(const T* base, long long elems) {
    const long long bytes = elems * (long long)sizeof(T);
    const unsigned range = (unsigned)(bytes < kMaxRange ? bytes : kMaxRange);
    return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, range, 0x00020000);
}

typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));

template <typename T>
struct Pair {
    T a, b;
};

template <typename T>
__device__ __forceinline__ Pair<T> load2(rsrc_t r, unsigned voff, unsigned soff) {
    if constexpr (sizeof(T) == 8) {
        return __builtin_bit_cast(Pair<T>, (v4u)__builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
    } else {
        return __builtin_bit_cast(Pair<T>, (v2u)__builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
    }
}
template <typename T>
__device__ __forceinline__ void store2(rsrc_t r, unsigned voff, unsigned soff, T a, T b) {
    const Pair<T> p{a, b};
    if constexpr (sizeof(T) == 8)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, p), r, voff, soff, 0);
    else
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u, p), r, voff, soff, 0);
}
template <typename T>
__device__ __forceinline__ void store1(rsrc_t r, unsigned voff, unsigned soff, T a) {
    if constexpr (sizeof(T) == 8)
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u, a), r, voff, soff, 0);
    else
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, a), r, voff, soff, 0);
}

// The value of the lane before (WEST) or after this one; zero at the wavefront's ends.
template <bool WEST>
__device__ __forceinline__ int lane_move(int x) {
    return __builtin_amdgcn_update_dpp(0, x, WEST ? 0x138 : 0x130, 0xf, 0xf, true);
}
template <bool WEST, typename T>
__device__ __forceinline__ T from_lane(T x) {
    if constexpr (sizeof(T) == 8) {
        struct W {
            int lo, hi;
        };
        const W w = __builtin_bit_cast(W, x);
        return __builtin_bit_cast(T, W{lane_move<WEST>(w.lo), lane_move<WEST>(w.hi)});
    } else {
        return __builtin_bit_cast(T, lane_move<WEST>(__builtin_bit_cast(int, x)));
    }
}

// Row tables are read with a wavefront-uniform index and never written by a
// pass: scalar loads from the constant address space.
typedef const __attribute__((address_space(4))) double* CTab;
typedef double ZRow __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(4))) ZRow* CRow;
__device__ __forceinline__ CTab ctab(const double* p) { return (CTab)(unsigned long long)p; }

// What a pass reads as its input iterate: nothing (zero with a zero ring), the
// Dirichlet ring of u_in around a zero interior, or u_in.
enum InputMode { kInZero = 0, kInRing = 1, kInFull = 2 };

// IN, XP (adds the prolongated coarse correction to the rows it consumes),
// DOWN (residual and restriction, else the optional residual norm), ZC (the
// coarse level is coarsened in z).
template <typename T, int NU, int IN, bool XP, bool DOWN, bool ZC, int COEF>
struct Pass {
    static constexpr bool ROWS = COEF == kRowTables;
    static constexpr int H = 2 * NU;
    static constexpr int U = 2;          // steps per group; rows in flight ahead of the consumed one
    static constexpr int N = H + 2 + U;  // rows held: row x0 + U - 1 - k in slot k
    // coefficients of a step's rows: the band's, the band's with the rows
    // outside it formed from their tables, or every row's from its tables
    static constexpr int kBand = 0, kMixed = 1, kTables = 2;
    // outputs of a step's rows: none of them in the chunk, all, or checked
    static constexpr int kNone = 0, kAll = 1, kCheck = 2;

    static_assert(H + 3 <= kRowPad, "rows a pass looks up beyond the level's");

    const PassArgs<T>& a;
    int p, za, zb, s, lend, nz;
    double lam;
    T om[2];
    bool act[2], own;
    CoefT<T> cu[2];
    double rw[ROWS ? 2 : 1], re[ROWS ? 2 : 1], rb[ROWS ? 2 : 1], rm[ROWS ? 2 : 1];  // radial tables
    int ic[2];                          // the columns, or an interior one in place of a column outside
    rsrc_t ru, rf, ro, rc_, re_;
    CRow zrow;
    CTab zct, zst, znt, pwl, pwr, rwm, rwp;
    unsigned rowb, crowb;               // bytes per row, fine and coarse
    unsigned voff, vring, vout, vec_, vfc;  // lane offsets: loads, ring-only loads, u store, e load, fc store
    T w1a, w1b, w2a, w2b;               // radial prolongation of the two columns from the pair (e_a, e_b)
    T wrm, wrp;                         // radial restriction at the coarse column under 2t
    T u[N][2], f[N][2];
    static constexpr int kRing = N <= 8 ? 8 : N <= 16 ? 16 : 32;
    T* ivl;                             // inverse diagonals of the rows held, [kRing][2][64]: row y in y % kRing
    Pair<T> pu[U], pf[U], pe[U];
    T ea[2];                            // radially interpolated coarse row at or below the consumed row
    T rs[2], r1[2];                     // restriction: the sum so far, the row below the next coarse row
    double acc;

    __device__ __forceinline__ explicit Pass(const PassArgs<T>& args) : a(args) {}

    __device__ __forceinline__ bool interior(int y) const { return y >= 1 && y <= nz - 2; }
    // rows that the band's coefficients serve; rows outside the interior keep
    // their values whatever the coefficients
    __device__ __forceinline__ bool regular(int y) const { return (y >= a.reg_lo && y < a.reg_hi) || !interior(y); }
    __device__ __forceinline__ int row(int y) const { return min(max(y, 0), nz - 1); }

    __device__ __forceinline__ unsigned ivpos(int y, int c) const {
        return ((unsigned)(y & (kRing - 1)) * 2 + c) * 64 + threadIdx.x;
    }

    // Radial interpolation of a loaded coarse pair to the lane's two columns.
    __device__ __forceinline__ void interpolate(const Pair<T>& e, T (&o)[2]) const {
#pragma clang fp contract(off)
        o[0] = fma(w1b, e.b, w1a * e.a);
        o[1] = fma(w2b, e.b, w2a * e.a);
    }
    __device__ __forceinline__ Pair<T> load_coarse(int K) const {
        return load2<T>(re_, vec_, (unsigned)min(max(K, 0), a.vc.nz - 1) * crowb);
    }

    __device__ __forceinline__ bool setup() {
        const LevelView& v = a.v;
        nz = v.nz;
        const int per = a.nchunks * a.nstrips;
        const int b = blockIdx.x;
        int q;
        if (a.xcd_major) {
            const int idx = b >> 3;
            p = a.p0 + (idx / per) * 8 + (b & 7);
            q = idx % per;
        } else {
            p = a.p0 + b / per;
            q = b % per;
        }
        if (a.mask && a.mask[p] == 0) return false;  // a frozen plane keeps its iterate
        const int chunk = q / a.nstrips, strip = q % a.nstrips;
        const int lane = threadIdx.x;
        const int t0 = strip * strip_step(NU), t = t0 + lane;
        const int c1 = 2 * t, c2 = 2 * t + 1;
        own = (strip == 0 || lane > NU) && (strip == a.nstrips - 1 || lane < 63 - NU);
        act[0] = c1 >= 1 && c1 <= v.nr - 2;
        act[1] = c2 <= v.nr - 2;
        za = 1 + chunk * a.chunk;
        zb = min(nz - 1, za + a.chunk);
        s = max(0, za - (H + 2)) & ~1;
        lend = min(nz - 1, zb + H + 1);
        lam = a.lam[p];
        // a column outside the plane's interior keeps its value: factor 0 and
        // finite coefficients
        om[0] = act[0] ? (T)a.omega : T(0);
        om[1] = act[1] ? (T)a.omega : T(0);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            ic[c] = act[c] ? (c == 0 ? c1 : c2) : 1;
            if constexpr (ROWS) {
                rw[c] = v.rw[ic[c]];
                re[c] = v.re[ic[c]];
                rb[c] = v.rb[ic[c]];
                rm[c] = v.rm[ic[c]];
            } else {
                const int i = ic[c];
                cu[c] = coef_as<T>(make_coef(v.rw[i], v.re[i], v.rb[i], v.rm[i], a.zc0, a.zs0, a.zn0, lam));
            }
        }
        // buffers from the chunk's first row on; rows are offsets from row s
        const long long first = (long long)p * v.pstride + (long long)s * v.pitch;
        const long long left = (long long)(nz - s) * v.pitch;
        rowb = (unsigned)(v.pitch * sizeof(T));
        if (IN != kInZero) ru = make_rsrc(a.u_in + first, left);
        rf = make_rsrc(a.f + first, left);
        ro = make_rsrc(a.u_out + first, left);
        const bool any = act[0] || act[1];
        voff = c1 < v.nr ? (unsigned)(c1 * sizeof(T)) : kOff;
        vring = any && act[0] && act[1] ? kOff : voff;
        vout = own && any ? voff : kOff;
        zrow = (CRow)(unsigned long long)a.zrow;
        zct = ctab(v.zc);
        zst = ctab(v.zs);
        znt = ctab(v.zn);
        if (XP || DOWN) crowb = (unsigned)(a.vc.pitch * sizeof(T));
        const int e0 = a.rc ? t : c1;  // first coarse column of the lane's pair
        if (XP) {
            re_ = make_rsrc(a.ec + (long long)p * a.vc.pstride, (long long)a.vc.nz * a.vc.pitch);
            vec_ = e0 < a.vc.nr ? (unsigned)(e0 * sizeof(T)) : kOff;
            w1a = T(1);
            w1b = T(0);
            w2a = (T)(act[1] && a.rc ? a.tr.pwl[c2] : 0.0);
            w2b = (T)(act[1] ? (a.rc ? a.tr.pwr[c2] : 1.0) : 0.0);
            pwl = ctab(a.tz.pwl);
            pwr = ctab(a.tz.pwr);
        }
        if (DOWN) {
            rc_ = make_rsrc(a.fc + (long long)p * a.vc.pstride, (long long)a.vc.nz * a.vc.pitch);
            const bool in = own && e0 >= 1 && e0 <= a.vc.nr - 2;
            vfc = (a.rc ? in : own && any) ? (unsigned)(e0 * sizeof(T)) : kOff;
            wrm = (T)(a.rc && in ? a.tr.rwm[e0] : 0.0);
            wrp = (T)(a.rc && in ? a.tr.rwp[e0] : 0.0);
            rwm = ctab(a.tz.rwm);
            rwp = ctab(a.tz.rwp);
        }
#pragma unroll
        for (int k = 0; k < N; ++k)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                u[k][c] = f[k][c] = T(0);
            }
        rs[0] = rs[1] = r1[0] = r1[1] = T(0);
        acc = 0.0;
        return true;
    }

    // Loads of row x into its parity's slot (rows beyond the chunk's last one
    // read that row again; they are never used).
    template <int J>
    __device__ __forceinline__ void issue(int x) {
        const int xr = min(x, lend);
        const unsigned so = (unsigned)(xr - s) * rowb;
        if (IN == kInFull)
            pu[J] = load2<T>(ru, voff, so);
        else if (IN == kInRing)  // lanes without a ring column read nothing on interior rows
            pu[J] = load2<T>(ru, interior(xr) ? vring : voff, so);
        pf[J] = load2<T>(rf, voff, so);
    }

    template <int J, bool PRED>
    __device__ __forceinline__ void consume(int x) {
#pragma clang fp contract(off)
        constexpr int B = U - 1 - J;
        const bool in = !PRED || interior(x);
        T v[2] = {T(0), T(0)};
        if (IN != kInZero) {
            v[0] = pu[J].a;
            v[1] = pu[J].b;
            if (IN == kInRing) {
                v[0] = in && act[0] ? T(0) : v[0];
                v[1] = in && act[1] ? T(0) : v[1];
            }
        }
        if (XP) {
            if (ZC) {
                if (J & 1) {  // odd row: between coarse rows (x - 1) / 2 and (x + 1) / 2
                    T eb[2];
                    interpolate(pe[J], eb);
                    const T wl = in ? (T)pwl[row(x)] : T(0), wr = in ? (T)pwr[row(x)] : T(0);
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        v[c] = v[c] + fma(wr, eb[c], wl * ea[c]);
                        ea[c] = eb[c];
                    }
                    pe[J] = load_coarse((x + 3) >> 1);
                } else {  // even row: on coarse row x / 2 (zero where that is the ring)
                    v[0] = v[0] + ea[0];
                    v[1] = v[1] + ea[1];
                }
            } else {
                T eb[2];
                interpolate(pe[J], eb);
                v[0] = v[0] + eb[0];
                v[1] = v[1] + eb[1];
                pe[J] = load_coarse(x + U);
            }
        }
        u[B][0] = v[0];
        u[B][1] = v[1];
        f[B][0] = act[0] ? pf[J].a : T(0);  // ring entries of f are the caller's and not read
        f[B][1] = act[1] ? pf[J].b : T(0);
        if constexpr (ROWS) {
            const ZRow z = zrow[x];
#pragma unroll
            for (int c = 0; c < 2; ++c)
                ivl[ivpos(x, c)] = (T)make_coef(rw[c], re[c], rb[c], rm[c], z.x, z.y, z.z, lam).invd;
        }
        issue<J>(x + U);
    }

    // Coefficients of column C in row y (slot K).
    template <int K, int C, int CM>
    __device__ __forceinline__ CoefT<T> coef(int y) const {
        if (CM == kBand) return cu[C];
        if constexpr (ROWS) {
            const ZRow z = zrow[y];
            Coef c = make_coef_products(rw[C], re[C], rb[C], rm[C], z.x, z.y, z.z, lam);
            CoefT<T> o = coef_as<T>(c);
            o.invd = ivl[ivpos(y, C)];
            return o;
        } else {
            const int r = row(y), i = ic[C];
            const LevelView& v = a.v;
            // the few rows outside the band read the radial tables again: kept
            // in registers they would cost every step 32 of them
            __asm__ volatile("" ::: "memory");
            return coef_as<T>(make_coef(v.rw[i], v.re[i], v.rb[i], v.rm[i], zct[r], zst[r], znt[r], lam));
        }
    }

    // One step (row x = x0 + J, x0 even).  PRED: rows of the ring, or beyond
    // it, may be among the step's rows and keep their values.
    template <int J, bool PRED, int CM, int OUT>
    __device__ __forceinline__ void step(int x) {
#pragma clang fp contract(off)
        constexpr int B = U - 1 - J;
        // every half-sweep of a step relaxes the columns of parity x - 1: the
        // lane's column C, whose far neighbour is the next (C = 1) or the
        // previous lane's other column, unchanged in this step
        constexpr int C = (J & 1) ? 0 : 1;
        T nb[H];
#pragma unroll
        for (int h = 0; h < H; ++h) nb[h] = from_lane<C == 0>(u[B + 1 + h][1 - C]);
        constexpr int R = B + H + 1;  // slot of the residual row
        constexpr bool RES = OUT != kNone;
        T rnw = T(0), rne = T(0);
        if (RES) {
            rnw = from_lane<true>(u[R][1]);
            rne = from_lane<false>(u[R][0]);
        }
        consume<J, PRED>(x);
        // each step loads its rows' tables: kept from step to step they would
        // be more scalar registers than there are
        if (ROWS) __asm__ volatile("" : "+s"(zrow));
        sweeps<0, J, PRED, CM>(x, nb);
        const int yf = x - H;  // final now
        if (OUT == kAll || (OUT == kCheck && yf >= za && yf < zb))
            store2<T>(ro, vout, (unsigned)(yf - s) * rowb, u[B + H][0], u[B + H][1]);
        if (!RES) return;
        const int y = yf - 1;
        if (DOWN) {
            T r0[2];
            residuals<J, PRED, CM>(y, rnw, rne, r0);
            if (!ZC) {
                if (OUT == kAll || (y >= za && y < zb)) restrict_row(y, r0[0], r0[1]);
            } else if (J & 1) {
                // y lies on coarse row y / 2: its own and the lower row's part
                const T wm = (T)rwm[row(y) >> 1];
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    rs[c] = fma(wm, r1[c], r0[c]);
                }
            } else {
                const int K = (y - 1) >> 1;
                if (OUT == kAll || (y - 1 >= za && y - 1 < zb)) {
                    const T wp = (T)rwp[K];
                    restrict_row(K, fma(wp, r0[0], rs[0]), fma(wp, r0[1], rs[1]));
                }
                r1[0] = r0[0];
                r1[1] = r0[1];
            }
        } else if (a.partial) {
            if (OUT == kAll || (y >= za && y < zb)) {
                T r0[2];
                residuals<J, PRED, CM>(y, rnw, rne, r0);
                const double d0 = own && act[0] ? (double)r0[0] : 0.0;
                const double d1 = own && act[1] ? (double)r0[1] : 0.0;
                acc = fma(d0, d0, acc);
                acc = fma(d1, d1, acc);
            }
        }
    }

    // Coarse right-hand side row K from the vertical sums of the lane's two
    // columns: the radial half of the restriction.
    __device__ __forceinline__ void restrict_row(int K, T v1, T v2) const {
        const unsigned so = (unsigned)K * crowb;
        if (a.rc)
            store1<T>(rc_, vfc, so, restrict3(from_lane<true>(v2), v1, v2, wrm, wrp));
        else
            store2<T>(rc_, vfc, so, act[0] ? v1 : T(0), act[1] ? v2 : T(0));
    }

    // Half-sweeps h, h + 1, ... of a step.
    template <int h, int J, bool PRED, int CM>
    __device__ __forceinline__ void sweeps(int x, const T (&nb)[H]) {
        if constexpr (h < H) {
            constexpr int C = (J & 1) ? 0 : 1, K = U - 1 - J + 1 + h;
            const int y = x - 1 - h;
            const T w = C == 0 ? nb[h] : u[K][0], e = C == 0 ? u[K][1] : nb[h];
            T n;
            if (CM == kMixed && regular(y))
                n = relax(u[K][C], f[K][C], w, e, u[K + 1][C], u[K - 1][C], cu[C], om[C]);
            else
                n = relax(u[K][C], f[K][C], w, e, u[K + 1][C], u[K - 1][C], coef<K, C, CM>(y), om[C]);
            u[K][C] = !PRED || interior(y) ? n : u[K][C];
            sweeps<h + 1, J, PRED, CM>(x, nb);
        }
    }

    template <int J, bool PRED, int CM>
    __device__ __forceinline__ void residuals(int y, T nw, T ne, T (&r)[2]) const {
        constexpr int K = U - 1 - J + H + 1;
        T x1, x2;
        if (CM == kMixed && regular(y)) {
            x1 = residual(u[K][0], f[K][0], nw, u[K][1], u[K + 1][0], u[K - 1][0], cu[0]);
            x2 = residual(u[K][1], f[K][1], u[K][0], ne, u[K + 1][1], u[K - 1][1], cu[1]);
        } else {
            x1 = residual(u[K][0], f[K][0], nw, u[K][1], u[K + 1][0], u[K - 1][0], coef<K, 0, CM>(y));
            x2 = residual(u[K][1], f[K][1], u[K][0], ne, u[K + 1][1], u[K - 1][1], coef<K, 1, CM>(y));
        }
        const bool in = !PRED || interior(y);
        r[0] = in ? x1 : T(0);
        r[1] = in ? x2 : T(0);
    }

    template <bool PRED, int CM, int OUT>
    __device__ __forceinline__ void group(int x0) {
        step<0, PRED, CM, OUT>(x0);
        step<1, PRED, CM, OUT>(x0 + 1);
#pragma unroll
        for (int k = N - 1; k >= U; --k)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                u[k][c] = u[k - U][c];
                f[k][c] = f[k - U][c];
            }
    }

    // The rows whose coefficients the group of steps from x0 uses are rows
    // max(x0 - H - 1, s) .. x0 + U - 2 (rows below s hold no values and feed
    // none that are used).  All interior, the prolongated rows included:
    __device__ __forceinline__ bool plain(int x0) const { return max(x0 - H - 1, s) >= 1 && x0 + U - 1 <= nz - 2; }
    // every interior one in the band
    __device__ __forceinline__ bool band(int x0) const {
        return max(max(x0 - H - 1, s), 1) >= a.reg_lo && min(x0 + U - 2, nz - 2) < a.reg_hi;
    }
    // no row of the group's outputs is in the chunk; all are
    __device__ __forceinline__ bool none(int x0) const { return x0 + U - 1 - H < za; }
    __device__ __forceinline__ bool all(int x0) const { return x0 - H - 2 >= za && x0 + U - 1 - H < zb; }

    __device__ __forceinline__ void run() {
        if (!setup()) return;
        if constexpr (ROWS) {
            __shared__ T ring[kRing * 2 * 64];
            ivl = ring;
        }
        issue<0>(s);
        issue<1>(s + 1);
        if (XP) {
            if (ZC) {
                interpolate(load_coarse(s >> 1), ea);
                pe[1] = load_coarse((s >> 1) + 1);
            } else {
                pe[0] = load_coarse(s);
                pe[1] = load_coarse(s + 1);
            }
        }
        // last step: the residual of row zb (down, coarsened in z) or zb - 1
        const int xlast = (DOWN && ZC ? zb : zb - 1) + H + 1;
        int x0 = s;
        if constexpr (ROWS) {
            for (; x0 <= xlast; x0 += U) {
                if (plain(x0) && none(x0))
                    group<false, kTables, kNone>(x0);
                else if (plain(x0) && all(x0))
                    group<false, kTables, kAll>(x0);
                else
                    group<true, kTables, kCheck>(x0);
            }
        } else {
            // the band's groups in a loop of their own between the others', so
            // that the others' registers are not its
            if (COEF == kSomeRows)
                for (; x0 <= xlast && !band(x0); x0 += U) group<true, kMixed, kCheck>(x0);
            for (; x0 <= xlast && (COEF == kOneBand || band(x0)); x0 += U) {
                if (plain(x0) && none(x0))
                    group<false, kBand, kNone>(x0);
                else if (plain(x0) && all(x0))
                    group<false, kBand, kAll>(x0);
                else
                    group<true, kBand, kCheck>(x0);
            }
            if (COEF == kSomeRows)
                for (; x0 <= xlast; x0 += U) group<true, kMixed, kCheck>(x0);
        }
        if (!DOWN && a.partial) {
            // fixed-order sum over the wavefront
#pragma unroll
            for (int w = 32; w > 0; w >>= 1) acc += __shfl_xor(acc, w);
            if (threadIdx.x == 0) {
                const int per = a.nchunks * a.nstrips;
                const int q = a.xcd_major ? (int)(blockIdx.x >> 3) % per : (int)blockIdx.x % per;
                a.partial[(long long)p * a.partial_ld + q] = acc;
            }
        }
    }
};

constexpr int kind_input(int k) { return k == kDownZero ? kInZero : k == kDownRing || k == kDownPro ? kInRing : kInFull; }

template <typename T, int NU, int KIND, bool ZC, int COEF>
using PassOf = Pass<T, NU, kind_input(KIND), (KIND >= kDownPro), (KIND != kUp), ZC, COEF>;

// Two wavefronts per SIMD (up to 256 registers) where that spills nothing or
// little, else one: the FP64 passes of five and six sweeps, and of four that
// read their iterate (`zero`: a pass that starts from zero).  Chunks are cut for
// this many: V(4,4) at 129 x 64 x 129 takes 411 us, and 517 when cut for two.
template <typename T>
constexpr int pass_waves(int nu, int coef, bool zero) {
    return sizeof(T) == 4 || nu <= 3 || (nu == 4 && (coef != kSomeRows || zero)) ? 2 : 1;
}

template <typename T, int NU, int KIND, bool ZC, int COEF>
__global__ void __launch_bounds__(64, pass_waves<T>(NU, COEF, KIND == kDownZero)) k_pass(PassArgs<T> a) {
    PassOf<T, NU, KIND, ZC, COEF> pass(a);
    pass.run();
}

// The same pass under its own symbol, launched for the finest level with the
// default sweep count, so that kernel traces and counters report the finest
// level apart from the coarser ones.
template <typename T, int NU, int KIND, bool ZC, int COEF>
__global__ void __launch_bounds__(64, 2) k_pass_fine(PassArgs<T> a) {
    PassOf<T, NU, KIND, ZC, COEF> pass(a);
    pass.run();
}

// The finest level's up pass of one V-cycle and down pass of the next in one
// stream of rows: the coarse correction is prolongated into the input as rows
// are consumed, then nu2 + nu1 sweeps run back to back (the red-black order of
// the two passes), then the residual and its restriction.  The node
// arithmetic is that of the two passes, so the iterate and the coarse
// right-hand side are bitwise theirs; the residual norm between the passes is
// not formed.
template <typename T, int NU, bool ZC, int COEF>
__global__ void __launch_bounds__(64, pass_waves<T>(NU, COEF, false)) k_pass_merge(PassArgs<T> a) {
    PassOf<T, NU, kMerge, ZC, COEF> pass(a);
    pass.run();
}

// ---- host side: launch shape and arguments ----

inline int strips_of(int nr, int nu) {
    const int lanes = (nr - 1) / 2 + 1;  // column pairs, both ring columns included
    return lanes <= 64 ? 1 : 1 + (lanes - 64 + strip_step(nu) - 1) / strip_step(nu);
}

// Launch shape of a pass with nu sweeps on level l.
template <typename T>
Shape pass_shape(const cylpoisson_plan* p, int l, int nu, bool down, bool merge = false) {
    const DeviceLevel& L = p->dl[l];
    Shape sh;
    sh.nstrips = strips_of(L.v.nr, nu);
    const int outside = L.v.nz - 2 - (L.reg_hi - L.reg_lo);
    // other sweep counts than the default's two (four merged) have one form
    sh.coef = nu != (merge ? 4 : 2) ? kSomeRows
              : outside <= 0        ? kOneBand
              : merge || outside > kFewRows ? kRowTables
                                            : kSomeRows;
    const int rows = L.v.nz - 2;
    int chunk = merge ? p->opt.chunk_rows_merge : l == 0 ? p->opt.chunk_rows : p->opt.chunk_rows_coarse;
    const bool automatic = chunk <= 0;
    // beside other solves fewer; but the finest FP64 up pass leaves the norms'
    // partial sums, whose order must be that of a solve alone
    const int share = l == 0 && !down && sizeof(T) == 8 ? 1 : p->share;
    // (a coarser level's down pass starts from zero)
    const int waves = pass_waves<T>(nu, sh.coef, down && !merge && l > 0);
    if (automatic) {
        // as many chunks as keep every wavefront resident at once
        auto rows_for = [&](int n) {
            const int per_plane = std::max(1, n / (share * p->nt * sh.nstrips));
            return std::max(kMinChunk, (rows + per_plane - 1) / per_plane);
        };
        chunk = rows_for(kPassWaves * waves / 2);
        // A merged chunk of c rows runs c + 19 or so steps.  Where it is short, a
        // second wavefront a SIMD mostly repeats rows of the first: up to
        // kShortChunk rows with one, one it is (151 x 45 x 203, 10 rows or 19: 382
        // and 366 us the solve; 129 x 64 x 129, 8 or 16: 275 and 268; 101 x 64 x 401,
        // 13 or 25: 549 and 546; 400 x 128 x 512, 128 or 255: 2412 and 2522).
        if (merge && share == 1 && waves == 2) {
            const int longer = rows_for(kPassWaves / 2);
            if (longer <= kShortChunk) chunk = longer;
        }
    }
    // an up pass keeps one norm partial per wavefront: at most 64 a plane
    // (what a check reads back) unless the caller asked for more chunks than
    // that, never more than the partials' array holds
    if (!down) {
        const int kept = automatic || (rows + chunk - 1) / chunk <= kSlotPartial ? kSlotPartial : kMaxPartial;
        const int most = std::max(1, kept / sh.nstrips);
        chunk = std::max(chunk, (rows + most - 1) / most);
    }
    chunk = std::min(std::max(chunk, 1), std::max(rows, 1));
    sh.chunk = chunk;
    sh.nchunks = (rows + chunk - 1) / chunk;
    sh.per_plane = sh.nchunks * sh.nstrips;
    sh.zc = p->dl[l + 1].v.nz < L.v.nz;
    return sh;
}

// Arguments of a pass over planes p0 .. p0 + np - 1 (its grid is sh.per_plane * np).
template <typename T>
PassArgs<T> make_args(const cylpoisson_plan* p, int l, const Shape& sh, int p0, int np) {
    const DeviceLevel& L = p->dl[l];
    const DeviceLevel& C = p->dl[l + 1];
    PassArgs<T> a{};
    a.v = L.v;
    a.vc = C.v;
    a.tr = L.tr;
    a.tz = L.tz;
    a.lam = p->d_lam;
    a.zrow = L.zrow;
    a.rc = C.v.nr < L.v.nr ? 1 : 0;
    a.reg_lo = L.reg_lo;
    a.reg_hi = L.reg_hi;
    a.omega = p->opt.omega;
    a.zc0 = L.zc0;
    a.zs0 = L.zs0;
    a.zn0 = L.zn0;
    a.chunk = sh.chunk;
    a.nchunks = sh.nchunks;
    a.nstrips = sh.nstrips;
    a.p0 = p0;
    a.mask = p->mask_live ? p->d_mask : nullptr;
    a.xcd_major = (np % 8 == 0) ? 1 : 0;
    return a;
}

// The kernel of a pass: under the finest level's symbol for the default sweeps.
template <typename T, int NU, int KIND, bool ZC, int COEF>
hipError_t launch_one(bool fine, const PassArgs<T>& a, int blocks, hipStream_t s) {
    if constexpr (KIND == kMerge) {
        k_pass_merge<T, NU, ZC, COEF><<<blocks, 64, 0, s>>>(a);
    } else if constexpr (NU == 2) {
        // the finest level's ring is not zero; a coarser one's is
        if constexpr (KIND != kDownZero || sizeof(T) == 4)
            if (fine) {
                k_pass_fine<T, NU, KIND, ZC, COEF><<<blocks, 64, 0, s>>>(a);
                return hipGetLastError();
            }
        if constexpr (KIND == kDownRing)
            return hipErrorInvalidValue;
        else
            k_pass<T, NU, KIND, ZC, COEF><<<blocks, 64, 0, s>>>(a);
    } else {
        (void)fine;
        k_pass<T, NU, KIND, ZC, COEF><<<blocks, 64, 0, s>>>(a);
    }
    return hipGetLastError();
}

template <typename T, int NU, int KIND, int COEF>
hipError_t launch_zc(bool fine, const Shape& sh, const PassArgs<T>& a, int np, hipStream_t s) {
    return sh.zc ? launch_one<T, NU, KIND, true, COEF>(fine, a, sh.per_plane * np, s)
                 : launch_one<T, NU, KIND, false, COEF>(fine, a, sh.per_plane * np, s);
}

}  // namespace

}  // namespace cp
