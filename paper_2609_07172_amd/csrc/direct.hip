// Exact solve of one coarse level of the V-cycle (the coarsest level the
// V-cycle visits when this solve is active), for every Fourier plane.
//
// The mode operator of a level is separable (App. A: every face conductance
// is a radial table entry times an axial one), so on a level's interior
//   A_p = Zc (x) T_r(lambda_p) + T_z (x) R_b
// with Zc = diag(zc_k), R_b = diag(rb_i), the axial tridiagonal T_z
// (T_z[k][k] = zs_k + zn_k, off-diagonals -zs_k, -zn_k) and the radial
// tridiagonal T_r(lambda) (diagonal rw_i + re_i + lambda rm_i, off-diagonals
// -rw_i, -re_i); this is the same operator the point kernels apply
// (Eqs. interior_base_diagonal, matrix_free_mode_operator).  With the
// generalised eigenvectors T_z V = Zc V Sigma, V^T Zc V = I (computed on the
// host when the plan is built), A_p u = f becomes, for each axial eigenvector
// j, one tridiagonal system along r:
//   (T_r(lambda_p) + sigma_j R_b) w_j = (V^T f)_j,   u = V w.
// The transforms are dense contractions and run on the FP64 matrix cores
// (v_mfma_f64_16x16x4f64: D += A B with A 16 x 4, B 4 x 16; lane l holds
// A[l % 16][l / 16], B[l / 16][l % 16] and D[l / 16 + 4q][l % 16], q < 4), V and
// V^T packed in the A operand's lane order when the plan is built.  The
// eliminations use factors formed then too (per mode: their chain is a
// division a row), which leaves one fused multiply-add a row,
//   d_i = (rw_i m_i) d_{i-1} + m_i g_i,   w_i = (re_i m_i) w_{i+1} + d_i,
// and run as segmented recurrences: a lane takes four rows of one eigenvector,
// the segments of an eigenvector are neighbouring lanes, and the carry into
// each segment is a scan of their affine maps by cross-lane moves; the
// rows are then run again from the carry.  Rows past the last have m = 0, which
// makes them zero.
//
// Up to 64 interior nodes each way, one workgroup solves a plane with
// everything between the two transforms in LDS (k_direct).  Up to 128, a plane
// is more matrix work than one compute unit should do alone: k_direct_fwd
// takes 32 eigenvectors of a plane per workgroup and writes w to the level's r
// array (free where the V-cycle stops), k_direct_inv 32 axial rows.  The
// workgroups of a plane run on one XCD, whose L2 serves all but the first read
// of f and w.  The coarse correction of a V-cycle has a zero Dirichlet ring, so
// only interior values enter and only interior values are written.
//
// What bounds it: latency (a workgroup's loads, products, scan and stores
// follow one another) and, at 128 planes of 99 x 127, 7 us of the matrix cores
// a transform.  One workgroup per plane: 3.9 us at 16 planes of 15 x 15 (8.3
// with the products on the vector unit and one lane per eigenvector dividing
// its way along r), 13 us at 64 planes of 63 x 63 (33).  Two kernels: 10 + 9 us
// at 45 planes of 74 x 100 (18 + 12 in halves of a plane with one chain of a
// ninth of the rows per lane), 9 + 7 at 64 of 49 x 99 (14 + 9), 23 + 20 at 128 of
// 99 x 127 (26 + 18).

#include "direct_tile.h"

#include <algorithm>
#include <cmath>

namespace cp {

namespace {

template <typename T>
struct DirectArgs {
    LevelView v;          // the direct level
    const T* f;           // right-hand side (the level's f)
    T* u;                 // answer (the level's u; its ring stays zero)
    double* w;            // two-kernel form: w between the kernels, row j of a plane in its interior row j
    const double* V;      // A operands of V^T, [group][k-step][lane]
    const double* VT;     // A operands of V
    const double* M;      // elimination factors, [mode][group][row of segment][chain and segment]
    const int* mask;      // per plane: 0 = frozen, or nullptr
    int p0, np;           // planes p0 .. p0 + np - 1
    int nc;               // cosine planes (the sine planes after them repeat modes 1, 2, ...)
    int ks;               // k-steps of the packed operands
};

// One workgroup per plane, up to 16 G interior nodes each way: G x G wavefronts,
// wavefront (g, c) forms the 16 x 16 tile of group g and radial columns 16 c of
// each transform, and a lane one segment of one eigenvector between them.
template <int G, typename T>
__global__ void __launch_bounds__(64 * G * G) k_direct(DirectArgs<T> a) {
    constexpr int N = 16 * G, NSEG = 4 * G, KS = 4 * G, LD = N + 1;
    __shared__ double gs[N * LD];
    const LevelView& v = a.v;
    const int plane = a.p0 + blockIdx.x;
    if (a.mask && a.mask[plane] == 0) return;  // whole workgroup, before any barrier
    const int nzi = v.nz - 2, nri = v.nr - 2;
    const int t = threadIdx.x, wave = t >> 6, l = t & 63, kr = l >> 4, cl = l & 15;
    const int grp = wave / G, col = 16 * (wave % G) + cl;
    const size_t base = (size_t)plane * v.pstride + v.pitch + 1;  // interior (0, 0)
    const bool in = col < nri;
    T fv[KS];
    double fb[KS], va[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const int k = 4 * s + kr;
        // (FP32: no condition, see product())
        if constexpr (sizeof(T) == 8)
            fv[s] = in && k < nzi ? a.f[base + (size_t)k * v.pitch + col] : T(0);
        else
            fv[s] = a.f[base + (size_t)min(k, nzi - 1) * v.pitch + min(col, nri - 1)];
        va[s] = a.V[((size_t)grp * KS + s) * 64 + l];
    }
#pragma unroll
    for (int s = 0; s < KS; ++s) fb[s] = sizeof(T) == 8 || (in && 4 * s + kr < nzi) ? (double)fv[s] : 0.0;
    const int chain = t / NSEG, seg = t % NSEG;
    SegTables tb;
    tb.load(v, a.M + ((size_t)mode_of(plane, a.nc) * G + chain / 16) * (kSegRows * 16 * NSEG) + t % (16 * NSEG),
            16 * NSEG, seg);
    dbl4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < KS; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(va[s], fb[s], acc, 0, 0, 0);
#pragma unroll
    for (int q = 0; q < 4; ++q) gs[(16 * grp + kr + 4 * q) * LD + col] = acc[q];
    __syncthreads();
    {
        double g[kSegRows];
        double* row = gs + chain * LD + seg * kSegRows;
#pragma unroll
        for (int u = 0; u < kSegRows; ++u) g[u] = row[u];
        eliminate<NSEG>(tb, g, seg);
#pragma unroll
        for (int u = 0; u < kSegRows; ++u) row[u] = g[u];
    }
#pragma unroll
    for (int s = 0; s < KS; ++s) va[s] = a.VT[((size_t)grp * KS + s) * 64 + l];
    __syncthreads();
    acc = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < KS; ++s)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(va[s], gs[(4 * s + kr) * LD + col], acc, 0, 0, 0);
    if (!in) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int k = 16 * grp + kr + 4 * q;
        if (k < nzi) a.u[base + (size_t)k * v.pitch + col] = (T)acc[q];
    }
}

// ---- two-kernel form: up to 128 interior nodes each way ----

constexpr int kBigThreads = 512, kBigSegs = 32;  // eight column tiles; 16 chains of 32 segments
// Groups of 16 per workgroup.  One alone (operands in registers) reads f and w
// twice as often: 37 + 27 us at 128 planes of 99 x 127 against 23 + 20, 14 + 10
// against 10 + 9 at 45 planes of 74 x 100; four (one workgroup per compute unit,
// no other to overlap its phases) 24 + 23 and 15 + 13.
constexpr int kBigE = 2;

// Workgroup -> (plane, first group); the workgroups of one plane are dealt to
// one of the eight XCDs.  False for the padding workgroups of the last eight
// planes.
__device__ __forceinline__ bool big_block(int groups, int np, int* plane, int* g) {
    const int idx = (int)blockIdx.x >> 3, per = (groups + kBigE - 1) / kBigE;
    *plane = (idx / per) * 8 + ((int)blockIdx.x & 7);
    *g = (idx % per) * kBigE;
    return *plane < np;
}

// The products of a workgroup's groups: B operands src[k * pitch + col], k < n,
// in registers and the A operands in LDS (`as`, kBigE ks 64 values), where
// every wavefront reads them, all loaded at once.  Every thread of the
// workgroup calls it; wavefronts past the last column tile (!on) only stage.
template <int KS, typename S>
__device__ __forceinline__ void product(const double* __restrict__ A, int ks, int groups, int g0, double* as,
                                        const S* __restrict__ src, size_t pitch, int n, int col, int cols, bool on,
                                        int l, dbl4 (&acc)[kBigE]) {
    constexpr int NA = (kBigE * KS * 32 + kBigThreads - 1) / kBigThreads;  // 16-byte pieces per thread
    const double2* ag = reinterpret_cast<const double2*>(A + (size_t)g0 * ks * 64);
    S fv[KS];
    double2 st[NA];
    // pieces past the last group's repeat its last one
    const int pieces = min(kBigE, groups - g0) * ks * 32;
#pragma unroll
    for (int i = 0; i < NA; ++i) st[i] = ag[min((int)threadIdx.x + i * kBigThreads, pieces - 1)];
    if constexpr (sizeof(S) == 8) {
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int k = 4 * s + (l >> 4);
            fv[s] = col < cols && k < n ? src[(size_t)k * pitch + col] : S(0);
        }
    } else if (on) {
        // A load under a condition, converted, waits for itself (64 planes of
        // 127 x 127: 21.6 us the forward kernel, 14.5 so), so rows and columns past
        // the last repeat it and are dropped below.  In FP64, without the
        // conversion, this costs the inverse kernel 1 us of its 20.5.
        const S* at = src + min(col, cols - 1);
#pragma unroll
        for (int s = 0; s < KS; ++s) fv[s] = at[(size_t)min(4 * s + (l >> 4), n - 1) * pitch];
    }
#pragma unroll
    for (int i = 0; i < NA; ++i)
        reinterpret_cast<double2*>(as)[min((int)threadIdx.x + i * kBigThreads, pieces - 1)] = st[i];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kBigE; ++e) acc[e] = dbl4{0.0, 0.0, 0.0, 0.0};
    if (!on) return;
    double fb[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s)
        fb[s] = sizeof(S) == 8 || (col < cols && 4 * s + (l >> 4) < n) ? (double)fv[s] : 0.0;
    // (a group past the last multiplies the staging of the one before it or
    // what the LDS held: its results are not used)
#pragma unroll
    for (int s = 0; s < KS; ++s)
        if (s < ks)
#pragma unroll
            for (int e = 0; e < kBigE; ++e)
                acc[e] = __builtin_amdgcn_mfma_f64_16x16x4f64(as[((size_t)min(e, groups - 1 - g0) * ks + s) * 64 + l],
                                                              fb[s], acc[e], 0, 0, 0);
}

// Transform and eliminations of 32 eigenvectors.
template <int KS, typename T>
__global__ void __launch_bounds__(kBigThreads, 4) k_direct_fwd(DirectArgs<T> a) {
    constexpr int LD = kDirectBigMax + 1;
    __shared__ double gs[16 * kBigE * LD];
    __shared__ __attribute__((aligned(16))) double as[kBigE * KS * 64];
    const LevelView& v = a.v;
    const int nzi = v.nz - 2, nri = v.nr - 2;
    const int groups = (nzi + 15) / 16;
    int pl, g0;
    if (!big_block(groups, a.np, &pl, &g0)) return;  // whole workgroup
    const int plane = a.p0 + pl;
    if (a.mask && a.mask[plane] == 0) return;  // whole workgroup, before any barrier
    const int t = threadIdx.x, wave = t >> 6, l = t & 63;
    const int col = 16 * wave + (l & 15);
    const int chain = t / kBigSegs, seg = t % kBigSegs;
    {
        dbl4 acc[kBigE];
        product<KS>(a.V, a.ks, groups, g0, as, a.f + (size_t)plane * v.pstride + v.pitch + 1, v.pitch, nzi, col,
                    nri, 16 * wave < nri, l, acc);
        if (16 * wave < nri)
#pragma unroll
            for (int e = 0; e < kBigE; ++e)
#pragma unroll
                for (int q = 0; q < 4; ++q) gs[(16 * e + (l >> 4) + 4 * q) * LD + col] = acc[e][q];
    }
    SegTables tb[kBigE];
#pragma unroll
    for (int e = 0; e < kBigE; ++e)
        tb[e].load(v, a.M + ((size_t)mode_of(plane, a.nc) * groups + min(g0 + e, groups - 1)) * (kSegRows * kBigThreads) + t,
                   kBigThreads, seg);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kBigE; ++e) {
        const int j = 16 * (g0 + e) + chain;
        double g[kSegRows];
#pragma unroll
        for (int u = 0; u < kSegRows; ++u) {
            const int i = seg * kSegRows + u;
            g[u] = i < nri ? gs[(16 * e + chain) * LD + i] : 0.0;
        }
        eliminate<kBigSegs>(tb[e], g, seg);
        if (j < nzi) {
            double* wout = a.w + (size_t)plane * v.pstride + (size_t)(j + 1) * v.pitch + 1 + seg * kSegRows;
#pragma unroll
            for (int u = 0; u < kSegRows; ++u)
                if (seg * kSegRows + u < nri) wout[u] = g[u];
        }
    }
}

// Inverse transform of 32 axial rows.
template <int KS, typename T>
__global__ void __launch_bounds__(kBigThreads, 4) k_direct_inv(DirectArgs<T> a) {
    __shared__ __attribute__((aligned(16))) double as[kBigE * KS * 64];
    const LevelView& v = a.v;
    const int nzi = v.nz - 2, nri = v.nr - 2;
    const int groups = (nzi + 15) / 16;
    int pl, g0;
    if (!big_block(groups, a.np, &pl, &g0)) return;
    const int plane = a.p0 + pl;
    if (a.mask && a.mask[plane] == 0) return;
    const int wave = threadIdx.x >> 6, l = threadIdx.x & 63;
    const int col = 16 * wave + (l & 15);
    dbl4 acc[kBigE];
    product<KS>(a.VT, a.ks, groups, g0, as, a.w + (size_t)plane * v.pstride + v.pitch + 1, v.pitch, nzi, col,
                nri, 16 * wave < nri, l, acc);
    if (col >= nri) return;
    T* u = a.u + (size_t)plane * v.pstride + v.pitch + 1;
#pragma unroll
    for (int e = 0; e < kBigE; ++e)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = 16 * (g0 + e) + (l >> 4) + 4 * q;
            if (k < nzi) u[(size_t)k * v.pitch + col] = (T)acc[e][q];
        }
}

// Eigenvalues and orthonormal eigenvectors of the symmetric n x n matrix S
// (row-major, overwritten) by cyclic Jacobi rotations: Q[k * n + j] is
// component k of eigenvector j, sig[j] its eigenvalue.  On a cache line's
// boundary: the rotations' loops are most of a plan's preparation (257 x 64 x 257:
// 22.4 ms; 26.0 where what is linked before them left the function 16 bytes off).
__attribute__((noinline, aligned(64))) void jacobi_eigen(int n, std::vector<double>& S, std::vector<double>& Q, std::vector<double>& sig) {
    Q.assign((size_t)n * n, 0.0);
    for (int k = 0; k < n; ++k) Q[(size_t)k * n + k] = 1.0;
    auto at = [&](int r, int c) -> double& { return S[(size_t)r * n + c]; };
    double scale = 0.0;
    for (int k = 0; k < n; ++k) scale = std::max(scale, std::fabs(at(k, k)));
    for (int sweep = 0; sweep < 100; ++sweep) {
        double off = 0.0;
        for (int r = 0; r < n; ++r)
            for (int c = r + 1; c < n; ++c) off = std::max(off, std::fabs(at(r, c)));
        if (off <= 1e-17 * scale) break;
        for (int r = 0; r < n; ++r)
            for (int c = r + 1; c < n; ++c) {
                const double arc = at(r, c);
                if (arc == 0.0) continue;
                // rotation in the (r, c) plane that zeroes S[r][c]
                const double theta = (at(c, c) - at(r, r)) / (2.0 * arc);
                const double tt = (theta >= 0.0 ? 1.0 : -1.0) / (std::fabs(theta) + std::sqrt(theta * theta + 1.0));
                const double cs = 1.0 / std::sqrt(tt * tt + 1.0), sn = tt * cs;
                for (int k = 0; k < n; ++k) {
                    const double skr = at(k, r), skc = at(k, c);
                    at(k, r) = cs * skr - sn * skc;
                    at(k, c) = sn * skr + cs * skc;
                }
                for (int k = 0; k < n; ++k) {
                    const double srk = at(r, k), sck = at(c, k);
                    at(r, k) = cs * srk - sn * sck;
                    at(c, k) = sn * srk + cs * sck;
                }
                for (int k = 0; k < n; ++k) {
                    const double qkr = Q[(size_t)k * n + r], qkc = Q[(size_t)k * n + c];
                    Q[(size_t)k * n + r] = cs * qkr - sn * qkc;
                    Q[(size_t)k * n + c] = sn * qkr + cs * qkc;
                }
                at(r, c) = at(c, r) = 0.0;  // zero in exact arithmetic
            }
    }
    sig.resize(n);
    for (int j = 0; j < n; ++j) sig[j] = at(j, j);
}

}  // namespace

bool direct_level_ok(const HostLevel& H, int max_nodes) {
    const int nzi = H.nz - 2, nri = H.nr - 2;
    if (nzi < 1 || nri < 1 || nzi > max_nodes || nri > max_nodes) return false;
    for (int k = 1; k <= nzi; ++k) {
        if (!(H.zc[k] > 0.0)) return false;
        // the axial operator must be symmetric for the eigenvector transform
        if (k < nzi) {
            const double a = H.zn[k], b = H.zs[k + 1];
            if (std::fabs(a - b) > 1e-12 * std::max(std::fabs(a), std::fabs(b))) return false;
        }
    }
    for (int i = 1; i <= nri; ++i)
        if (!(H.rb[i] > 0.0)) return false;
    return true;
}

void direct_tables(const HostLevel& H, std::vector<double>& V, std::vector<double>& sigma) {
    const int nzi = H.nz - 2;
    // S = Zc^-1/2 T_z Zc^-1/2 (symmetric); V = Zc^-1/2 Q, row-major [k][j]
    std::vector<double> S((size_t)nzi * nzi, 0.0), Q;
    for (int k = 0; k < nzi; ++k) {
        const int K = k + 1;
        S[(size_t)k * nzi + k] = (H.zs[K] + H.zn[K]) / H.zc[K];
        if (k + 1 < nzi) {
            const double off = -0.5 * (H.zn[K] + H.zs[K + 1]) / std::sqrt(H.zc[K] * H.zc[K + 1]);
            S[(size_t)k * nzi + k + 1] = off;
            S[(size_t)(k + 1) * nzi + k] = off;
        }
    }
    jacobi_eigen(nzi, S, Q, sigma);
    V.assign((size_t)nzi * nzi, 0.0);
    for (int k = 0; k < nzi; ++k)
        for (int j = 0; j < nzi; ++j) V[(size_t)k * nzi + j] = Q[(size_t)k * nzi + j] / std::sqrt(H.zc[k + 1]);
}

int direct_level(const cylpoisson_plan* p) {
    if (p->opt.direct == 1) return p->dir[0].level;
    if (p->opt.direct == 2) return p->dir[1].level;
    return -1;
}

bool direct_active(const cylpoisson_plan* p) { return direct_level(p) > 0; }

// Group size of the one-workgroup form: 16 G interior nodes each way.
int direct_g(const HostLevel& H) {
    const int n = std::max(H.nz, H.nr) - 2;
    return n <= 16 ? 1 : n <= 32 ? 2 : 4;
}

int direct_ksteps(const HostLevel& H, bool big) { return big ? (H.nz - 2 + 3) / 4 : 4 * direct_g(H); }

// Operand and factor tables of a level (zero padded), from its eigenvectors
// V [nzi][nzi], eigenvalues and the modes' shifts lam[0 .. nc - 1].
void direct_pack(const HostLevel& H, bool big, const std::vector<double>& V, const std::vector<double>& sigma,
                 const std::vector<double>& lam, int nc, std::vector<double>& Vp, std::vector<double>& VTp,
                 std::vector<double>& M) {
    const int nzi = H.nz - 2, nri = H.nr - 2;
    const int groups = big ? (nzi + 15) / 16 : direct_g(H), ks = direct_ksteps(H, big);
    Vp.assign((size_t)groups * ks * 64, 0.0);
    VTp = Vp;
    for (int g = 0; g < groups; ++g)
        for (int s = 0; s < ks; ++s)
            for (int l = 0; l < 64; ++l) {
                const int row = 16 * g + l % 16, k = 4 * s + l / 16;
                if (row >= nzi || k >= nzi) continue;
                const size_t at = ((size_t)g * ks + s) * 64 + l;
                Vp[at] = V[(size_t)k * nzi + row];   // (V^T)[row][k]
                VTp[at] = V[(size_t)row * nzi + k];  // V[row][k]
            }
    // elimination factors of (T_r(lambda) + sigma_j R_b) w = g along r:
    // m_i = 1 / (b_i - rw_i c_{i-1}), c_i = re_i m_i
    const int nseg = big ? kBigSegs : 4 * groups;
    const size_t per = (size_t)kSegRows * 16 * nseg;
    M.assign((size_t)nc * groups * per, 0.0);
    for (int q = 0; q < nc; ++q)
        for (int j = 0; j < nzi; ++j) {
            double* out = M.data() + ((size_t)q * groups + j / 16) * per + (size_t)(j % 16) * nseg;
            double c = 0.0;
            for (int i = 0; i < nri; ++i) {
                const int I = i + 1;
                const double b = H.rw[I] + H.re[I] + lam[q] * H.rm[I] + sigma[j] * H.rb[I];
                const double mi = 1.0 / (b - H.rw[I] * c);
                c = H.re[I] * mi;
                out[(size_t)(i % kSegRows) * 16 * nseg + i / kSegRows] = mi;
            }
        }
}

namespace {

template <int KS, typename T>
hipError_t launch_big(const DirectArgs<T>& a, hipStream_t s) {
    if constexpr (KS < 32)
        if (a.ks > KS) return launch_big<KS + 4, T>(a, s);
    const int groups = (a.v.nz - 2 + 15) / 16;
    const int blocks = 8 * ((a.np + 7) / 8) * ((groups + kBigE - 1) / kBigE);
    k_direct_fwd<KS><<<blocks, kBigThreads, 0, s>>>(a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_direct_inv<KS><<<blocks, kBigThreads, 0, s>>>(a);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_direct_t(cylpoisson_plan* p, const T* f, T* u, hipStream_t s, int p0, int np) {
    const DirectLevel& d = p->dir[p->opt.direct == 2 ? 1 : 0];
    const DeviceLevel& L = p->dl[d.level];
    if (np < 0) np = p->nt - p0;
    if (np <= 0) return hipSuccess;
    DirectArgs<T> a{};
    a.v = L.v;
    a.f = f;
    a.u = u;
    a.w = L.r;
    a.V = d.V;
    a.VT = d.VT;
    a.M = d.M;
    a.mask = p->mask_live ? p->d_mask : nullptr;
    a.p0 = p0;
    a.np = np;
    a.nc = p->nt / 2 + 1;
    const HostLevel& H = p->hl[d.level];
    a.ks = direct_ksteps(H, d.big);
    if (d.big) return launch_big<4, T>(a, s);
    switch (direct_g(H)) {
        case 1: k_direct<1, T><<<np, 64, 0, s>>>(a); break;
        case 2: k_direct<2, T><<<np, 256, 0, s>>>(a); break;
        default: k_direct<4, T><<<np, 1024, 0, s>>>(a); break;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_direct(cylpoisson_plan* p, hipStream_t s, int p0, int np) {
    const DeviceLevel& L = p->dl[direct_level(p)];
    return launch_direct_t<double>(p, L.f, L.u, s, p0, np);
}

hipError_t launch_direct32(cylpoisson_plan* p, hipStream_t s, int p0, int np) {
    const DeviceLevel32& L = p->dl32[direct_level(p)];
    return launch_direct_t<float>(p, L.f, L.u, s, p0, np);
}

}  // namespace cp
