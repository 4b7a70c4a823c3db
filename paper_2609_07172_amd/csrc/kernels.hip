// Reference HIP kernels for gfx950: one kernel per elementary multigrid step.
// They are the correctness baseline and serve the small levels; the fused
// streaming kernels (fused.hip) take over the large levels.
#include "cp_internal.h"
#include "stencil.h"

namespace cp {

namespace {

constexpr int kTx = 64, kTy = 4;
// Lines up to this length are solved by cyclic reduction in one workgroup.
constexpr int kMaxPcrLine = 1024;

// ---------------------------------------------------------------- DFT (FMA)
// Y[p][c] = cs(c) * sum_j M[p][j] X[j][c] for c in [0, ncols), p in [0, n).
// Each thread owns one column c and kDftRows consecutive output rows; the
// matrix row index is uniform across the wavefront, so M is read through the
// scalar unit.
constexpr int kDftRows = 16;

__global__ void __launch_bounds__(256) k_dft(const double* __restrict__ M,
                                             const double* __restrict__ X,
                                             double* __restrict__ Y, int n, long long ncols,
                                             const double* __restrict__ cs) {
    const long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const int p0 = blockIdx.y * kDftRows;
    if (c >= ncols) return;
    double acc[kDftRows];
#pragma unroll
    for (int q = 0; q < kDftRows; ++q) acc[q] = 0.0;
    const int rows = min(kDftRows, n - p0);
    for (int j = 0; j < n; ++j) {
        const double x = X[(long long)j * ncols + c];
        const double* m = M + (long long)p0 * n + j;
#pragma unroll
        for (int q = 0; q < kDftRows; ++q)
            if (q < rows) acc[q] = fma(m[(long long)q * n], x, acc[q]);
    }
    const double scale = cs ? cs[c] : 1.0;
#pragma unroll
    for (int q = 0; q < kDftRows; ++q)
        if (q < rows) Y[(long long)(p0 + q) * ncols + c] = acc[q] * scale;
}

// ------------------------------------------------------------ initialisation
// Fine-level iterate: zero interior; ring of plane 0 holds the Dirichlet data
// (axial faces win at corners), rings of the other planes are zero because a
// theta-invariant boundary has only an m = 0 component (Eq. mode_rhs).
__global__ void k_init_fine_u(LevelView v, double* u, double prz, double prout, double pz0,
                              double pzl) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int k = blockIdx.y * blockDim.y + threadIdx.y;
    const int p = blockIdx.z;
    if (i >= v.nr || k >= v.nz) return;
    double val = 0.0;
    if (p == 0) {
        if (i == 0) val = prz;
        if (i == v.nr - 1) val = prout;
        if (k == 0) val = pz0;
        if (k == v.nz - 1) val = pzl;
    }
    u[(long long)p * v.pstride + (long long)k * v.pitch + i] = val;
}

__global__ void k_zero_interior(LevelView v, double* u) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x + 1;
    const int k = blockIdx.y * blockDim.y + threadIdx.y + 1;
    const int p = blockIdx.z;
    if (i > v.nr - 2 || k > v.nz - 2) return;
    u[(long long)p * v.pstride + (long long)k * v.pitch + i] = 0.0;
}

__global__ void k_zero(double* p, long long n) {
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) p[t] = 0.0;
}

__global__ void k_copy_interior(LevelView v, const double* __restrict__ src, double* __restrict__ dst) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x + 1;
    const int k = blockIdx.y * blockDim.y + threadIdx.y + 1;
    const int p = blockIdx.z;
    if (i > v.nr - 2 || k > v.nz - 2) return;
    const long long o = (long long)p * v.pstride + (long long)k * v.pitch + i;
    dst[o] = src[o];
}

// --------------------------------------------------------- red-black sweep
// One colour of red-black over-relaxed Gauss-Seidel on A_p = A_0 + lambda_p M
// (Eq. matrix_free_mode_operator).  Colour = (i + k) & 1.  In place.
__global__ void __launch_bounds__(256) k_rb(LevelView v, const double* __restrict__ lam,
                                            double* __restrict__ u,
                                            const double* __restrict__ f, int color,
                                            double omega) {
    const int k = blockIdx.y * blockDim.y + threadIdx.y + 1;
    const int i = 2 - (color ^ (k & 1)) + 2 * (blockIdx.x * blockDim.x + threadIdx.x);
    const int p = blockIdx.z;
    if (i > v.nr - 2 || k > v.nz - 2) return;
    const long long o = (long long)p * v.pstride + (long long)k * v.pitch + i;
    const Coef c = coef_at(v, i, k, lam[p]);
    u[o] = relax(u[o], f[o], u[o - 1], u[o + 1], u[o - v.pitch], u[o + v.pitch], c, omega);
}

// ------------------------------------------------------- line relaxation
// Zebra line relaxation: every interior line of one colour is solved exactly
// with the lines of the other colour held fixed (line Gauss-Seidel), by the
// Thomas algorithm, one thread per line.  Along r, line k carries
//   -G_W u_{i-1} + (D0 + lambda mu) u_i - G_E u_{i+1} = f_i + G_S u_{k-1,i} + G_N u_{k+1,i}
// (the ring values enter the right-hand side at i = 1 and i = nr - 2); along z
// the roles of (W, E) and (S, N) swap.  The forward elimination keeps the
// modified super-diagonal c'_j in `scratch` and the modified right-hand side
// d'_j in the line's own entries of u (the exact line solve does not read
// them); back substitution then overwrites them with the solution.
__global__ void __launch_bounds__(64) k_rline(LevelView v, const double* __restrict__ lam, double* __restrict__ u,
                                              const double* __restrict__ f, double* __restrict__ scratch,
                                              int color) {
    const int k = 1 + color + 2 * (blockIdx.x * blockDim.x + threadIdx.x);
    const int p = blockIdx.y;
    if (k > v.nz - 2) return;
    const double l = lam[p];
    const long long row = (long long)p * v.pstride + (long long)k * v.pitch;
    double* ur = u + row;
    const double* fr = f + row;
    double* cr = scratch + row;
    const double* us = ur - v.pitch;
    const double* un = ur + v.pitch;
    const int ie = v.nr - 2;
    double cp = 0.0, dp = 0.0;
    for (int i = 1; i <= ie; ++i) {
        const Coef c = coef_at(v, i, k, l);
        double rhs = fma(c.gn, un[i], fma(c.gs, us[i], fr[i]));
        if (i == 1) rhs = fma(c.gw, ur[0], rhs);
        if (i == ie) rhs = fma(c.ge, ur[ie + 1], rhs);
        const double a = i > 1 ? c.gw : 0.0;  // the sub-diagonal is -a
        const double inv = 1.0 / fma(a, cp, c.diag);
        cp = (i < ie ? -c.ge : 0.0) * inv;
        dp = fma(a, dp, rhs) * inv;
        cr[i] = cp;
        ur[i] = dp;
    }
    double x = dp;
    for (int i = ie - 1; i >= 1; --i) {
        x = fma(-cr[i], x, ur[i]);
        ur[i] = x;
    }
}

__global__ void __launch_bounds__(64) k_zline(LevelView v, const double* __restrict__ lam, double* __restrict__ u,
                                              const double* __restrict__ f, double* __restrict__ scratch,
                                              int color) {
    const int i = 1 + color + 2 * (blockIdx.x * blockDim.x + threadIdx.x);
    const int p = blockIdx.y;
    if (i > v.nr - 2) return;
    const double l = lam[p];
    const long long col = (long long)p * v.pstride + i;
    double* uc = u + col;
    const double* fc = f + col;
    double* cc = scratch + col;
    const long long P = v.pitch;
    const int ke = v.nz - 2;
    double cp = 0.0, dp = 0.0;
    for (int k = 1; k <= ke; ++k) {
        const Coef c = coef_at(v, i, k, l);
        const long long o = (long long)k * P;
        double rhs = fma(c.ge, uc[o + 1], fma(c.gw, uc[o - 1], fc[o]));
        if (k == 1) rhs = fma(c.gs, uc[0], rhs);
        if (k == ke) rhs = fma(c.gn, uc[o + P], rhs);
        const double a = k > 1 ? c.gs : 0.0;
        const double inv = 1.0 / fma(a, cp, c.diag);
        cp = (k < ke ? -c.gn : 0.0) * inv;
        dp = fma(a, dp, rhs) * inv;
        cc[o] = cp;
        uc[o] = dp;
    }
    double x = dp;
    for (int k = ke - 1; k >= 1; --k) {
        const long long o = (long long)k * P;
        x = fma(-cc[o], x, uc[o]);
        uc[o] = x;
    }
}

// The same line solves with one workgroup per line and one thread per
// unknown, by parallel cyclic reduction in LDS: at stride s = 1, 2, 4, ...
// every equation eliminates its neighbours s positions away, so after
// ceil(log2 n) steps each equation holds its own unknown alone.  Each thread
// keeps its own pivot b and publishes 1/b, so a step costs one division.
// Lines run along r (ALONG_R, coalesced rows) or along z (one column).
// Consecutive lines go to one XCD (workgroups are dealt to the 8 XCDs in
// turn), so lines that share neighbour rows or cache lines share an L2.
template <bool ALONG_R>
__global__ void __launch_bounds__(1024) k_line_pcr(LevelView v, const double* __restrict__ lam,
                                                   double* __restrict__ u, const double* __restrict__ f,
                                                   int color, int lines) {
    extern __shared__ double sm[];
    const int n = ALONG_R ? v.nr - 2 : v.nz - 2;
    const int per_xcd = (lines + 7) / 8;
    const int j = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (j >= lines) return;  // whole workgroup: before any barrier
    const int line = 1 + color + 2 * j;
    const int p = blockIdx.y;
    const int t = threadIdx.x;
    const int m = blockDim.x;
    double* A = sm;
    double* I = sm + 2 * m;  // 1 / pivot
    double* C = sm + 4 * m;
    double* D = sm + 6 * m;
    const bool act = t < n;
    const int x = t + 1;
    const int i = ALONG_R ? x : line, k = ALONG_R ? line : x;
    const long long o = (long long)p * v.pstride + (long long)k * v.pitch + i;
    double a = 0.0, b = 1.0, c = 0.0, d = 0.0;
    if (act) {
        const Coef cf = coef_at(v, i, k, lam[p]);
        // neighbours across lines (held fixed) and the ring at the line's ends
        const double g_lo = ALONG_R ? cf.gw : cf.gs, g_hi = ALONG_R ? cf.ge : cf.gn;
        const long long step = ALONG_R ? 1 : v.pitch, across = ALONG_R ? v.pitch : 1;
        const double x_lo = ALONG_R ? cf.gs : cf.gw, x_hi = ALONG_R ? cf.gn : cf.ge;
        d = fma(x_hi, u[o + across], fma(x_lo, u[o - across], f[o]));
        if (x == 1) d = fma(g_lo, u[o - step], d);
        if (x == n) d = fma(g_hi, u[o + step], d);
        a = x > 1 ? -g_lo : 0.0;
        c = x < n ? -g_hi : 0.0;
        b = cf.diag;
    }
    int buf = 0;
    A[t] = a;
    I[t] = 1.0 / b;
    C[t] = c;
    D[t] = d;
    __syncthreads();
    for (int st = 1; st < n; st <<= 1) {
        const double* a0 = A + buf * m;
        const double* i0 = I + buf * m;
        const double* c0 = C + buf * m;
        const double* d0 = D + buf * m;
        if (act) {
            const int lo = t - st, hi = t + st;
            double na = 0.0, nc = 0.0;
            if (lo >= 0) {
                const double al = -a * i0[lo];
                na = al * a0[lo];
                b = fma(al, c0[lo], b);
                d = fma(al, d0[lo], d);
            }
            if (hi < n) {
                const double ga = -c * i0[hi];
                nc = ga * c0[hi];
                b = fma(ga, a0[hi], b);
                d = fma(ga, d0[hi], d);
            }
            a = na;
            c = nc;
        }
        buf ^= 1;
        A[buf * m + t] = a;
        I[buf * m + t] = 1.0 / b;
        C[buf * m + t] = c;
        D[buf * m + t] = d;
        __syncthreads();
    }
    if (act) u[o] = d * I[buf * m + t];
}

// ---------------------------------------------------------------- residual
__global__ void __launch_bounds__(256) k_residual(LevelView v, const double* __restrict__ lam,
                                                  const double* __restrict__ u,
                                                  const double* __restrict__ f,
                                                  double* __restrict__ r) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x + 1;
    const int k = blockIdx.y * blockDim.y + threadIdx.y + 1;
    const int p = blockIdx.z;
    if (i > v.nr - 2 || k > v.nz - 2) return;
    const long long o = (long long)p * v.pstride + (long long)k * v.pitch + i;
    const Coef c = coef_at(v, i, k, lam[p]);
    r[o] = residual(u[o], f[o], u[o - 1], u[o + 1], u[o - v.pitch], u[o + v.pitch], c);
}

// ------------------------------------------------------------- restriction
// f_c = P^T r (full weighting on the distance-weighted bilinear P).
__global__ void __launch_bounds__(256) k_restrict(LevelView vf, LevelView vc, Transfer1D tr,
                                                  Transfer1D tz, const double* __restrict__ r,
                                                  double* __restrict__ fc) {
    const int I = blockIdx.x * blockDim.x + threadIdx.x + 1;
    const int K = blockIdx.y * blockDim.y + threadIdx.y + 1;
    const int p = blockIdx.z;
    if (I > vc.nr - 2 || K > vc.nz - 2) return;
    const int fi = tr.cidx[I], fk = tz.cidx[K];
    const double* rp = r + (long long)p * vf.pstride + (long long)fk * vf.pitch + fi;
    const double wzm = tz.rwm[K], wzp = tz.rwp[K];
    double col[3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
        col[a] = restrict3(rp[a - 1 - vf.pitch], rp[a - 1], rp[a - 1 + vf.pitch], wzm, wzp);
    fc[(long long)p * vc.pstride + (long long)K * vc.pitch + I] =
        restrict3(col[0], col[1], col[2], tr.rwm[I], tr.rwp[I]);
}

// ------------------------------------------------------------ prolongation
// u_f += P e_c, or u_f = P e_c on the interior when !ADD (the coarse ring is zero).
template <bool ADD>
__global__ void __launch_bounds__(256) k_prolong(LevelView vf, LevelView vc, Transfer1D tr,
                                                 Transfer1D tz, const double* __restrict__ uc,
                                                 double* __restrict__ u) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x + 1;
    const int k = blockIdx.y * blockDim.y + threadIdx.y + 1;
    const int p = blockIdx.z;
    if (i > vf.nr - 2 || k > vf.nz - 2) return;
    const int I = tr.pidx[i], K = tz.pidx[k];
    const double* c0 = uc + (long long)p * vc.pstride + (long long)K * vc.pitch + I;
    const double e = prolong_value(c0, vc.pitch, tr.pwl[i], tr.pwr[i], tz.pwl[k], tz.pwr[k]);
    double* o = u + (long long)p * vf.pstride + (long long)k * vf.pitch + i;
    if (ADD)
        *o += e;
    else
        *o = e;
}

// -------------------------------------------------------- coarsest solve
// u += A_p^{-1} (f - A_p u) with the inverse precomputed on the host per plane;
// one block per plane.  Interior unknown q = (k-1)*(nr-2) + (i-1).
__global__ void __launch_bounds__(256) k_coarse_solve(LevelView v, const double* __restrict__ lam,
                                                      const double* __restrict__ cinv, int n,
                                                      const double* __restrict__ f,
                                                      double* __restrict__ u) {
    extern __shared__ double sres[];
    const int p = blockIdx.x;
    const int ni = v.nr - 2;
    double* up = u + (long long)p * v.pstride;
    const double* fp = f + (long long)p * v.pstride;
    for (int q = threadIdx.x; q < n; q += blockDim.x) {
        const int i = q % ni + 1, k = q / ni + 1;
        const long long o = (long long)k * v.pitch + i;
        const Coef c = coef_at(v, i, k, lam[p]);
        sres[q] = residual(up[o], fp[o], up[o - 1], up[o + 1], up[o - v.pitch], up[o + v.pitch], c);
    }
    __syncthreads();
    const double* Ci = cinv + (long long)p * n * n;
    double* scor = sres + n;
    for (int q = threadIdx.x; q < n; q += blockDim.x) {
        double s = 0.0;
        for (int t = 0; t < n; ++t) s = fma(Ci[(long long)q * n + t], sres[t], s);
        scor[q] = s;
    }
    __syncthreads();
    for (int q = threadIdx.x; q < n; q += blockDim.x) {
        const int i = q % ni + 1, k = q / ni + 1;
        up[(long long)k * v.pitch + i] += scor[q];
    }
}

// Dirichlet ring of the fine-level iterate(s): plane 0 holds the face values
// (axial faces win at corners), other planes zero (Eq. mode_rhs).
__global__ void k_init_ring(LevelView v, double* u, double* u2, double prz, double prout,
                            double pz0, double pzl) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    const int p = blockIdx.y;
    const int n_rows = 2 * v.nr, n_cols = 2 * (v.nz - 2);
    if (q >= n_rows + n_cols) return;
    int i, k;
    if (q < n_rows) {
        i = q % v.nr;
        k = q < v.nr ? 0 : v.nz - 1;
    } else {
        const int c = q - n_rows;
        k = 1 + c % (v.nz - 2);
        i = c < v.nz - 2 ? 0 : v.nr - 1;
    }
    double val = 0.0;
    if (p == 0) {
        if (i == 0) val = prz;
        if (i == v.nr - 1) val = prout;
        if (k == 0) val = pz0;
        if (k == v.nz - 1) val = pzl;
    }
    const long long o = (long long)p * v.pstride + (long long)k * v.pitch + i;
    u[o] = val;
    u2[o] = val;
}

// Copy the Dirichlet ring (boundary rows and columns) of every plane.
__global__ void k_copy_ring(LevelView v, const double* __restrict__ src, double* __restrict__ dst) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;  // index along the ring
    const int p = blockIdx.y;
    const int n_rows = 2 * v.nr, n_cols = 2 * (v.nz - 2);
    if (q >= n_rows + n_cols) return;
    int i, k;
    if (q < n_rows) {
        i = q % v.nr;
        k = q < v.nr ? 0 : v.nz - 1;
    } else {
        const int c = q - n_rows;
        k = 1 + c % (v.nz - 2);
        i = c < v.nz - 2 ? 0 : v.nr - 1;
    }
    const long long o = (long long)p * v.pstride + (long long)k * v.pitch + i;
    dst[o] = src[o];
}

dim3 grid_interior(const LevelView& v, int nt, int xdiv = 1) {
    const int ni = (v.nr - 2 + xdiv - 1) / xdiv, nk = v.nz - 2;
    return dim3((ni + kTx - 1) / kTx, (nk + kTy - 1) / kTy, nt);
}

}  // namespace

hipError_t launch_dft(const double* M, const double* X, double* Y, int n, long long ncols,
                      const double* colscale, hipStream_t s) {
    dim3 grid((unsigned)((ncols + 255) / 256), (n + kDftRows - 1) / kDftRows);
    k_dft<<<grid, 256, 0, s>>>(M, X, Y, n, ncols, colscale);
    return hipGetLastError();
}

hipError_t launch_init_fine_u(const DeviceLevel& L, int nt, const cylpoisson_bc& bc, hipStream_t s) {
    dim3 grid((L.v.nr + kTx - 1) / kTx, (L.v.nz + kTy - 1) / kTy, nt);
    k_init_fine_u<<<grid, dim3(kTx, kTy), 0, s>>>(L.v, L.u, bc.phi_r_in, bc.phi_r_out, bc.phi_z0,
                                                   bc.phi_zL);
    return hipGetLastError();
}

hipError_t launch_zero_interior(const DeviceLevel& L, int nt, double* u, hipStream_t s) {
    k_zero_interior<<<grid_interior(L.v, nt), dim3(kTx, kTy), 0, s>>>(L.v, u);
    return hipGetLastError();
}

hipError_t launch_zero(double* p, long long n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    k_zero<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(p, n);
    return hipGetLastError();
}

hipError_t launch_copy_interior(const DeviceLevel& L, int nt, const double* src, double* dst,
                                hipStream_t s) {
    k_copy_interior<<<grid_interior(L.v, nt), dim3(kTx, kTy), 0, s>>>(L.v, src, dst);
    return hipGetLastError();
}

hipError_t launch_rb_sweep(const DeviceLevel& L, int nt, const double* lam, double* u,
                           const double* f, int color, double omega, hipStream_t s) {
    k_rb<<<grid_interior(L.v, nt, 2), dim3(kTx, kTy), 0, s>>>(L.v, lam, u, f, color, omega);
    return hipGetLastError();
}

hipError_t launch_line_sweep(const DeviceLevel& L, int nt, const double* lam, double* u, const double* f,
                             double* scratch, bool along_r, int color, hipStream_t s) {
    const int lines = along_r ? L.v.nz - 2 : L.v.nr - 2;
    const int mine = (lines - color + 1) / 2;  // lines 1 + color, 3 + color, ...
    if (mine <= 0) return hipSuccess;
    const int len = along_r ? L.v.nr - 2 : L.v.nz - 2;
    if (len <= kMaxPcrLine) {
        // one workgroup per line: a power of two of threads covering the line
        int m = 64;
        while (m < len) m <<= 1;
        const size_t lds = 8 * (size_t)m * sizeof(double);
        const unsigned blocks = 8u * (unsigned)((mine + 7) / 8);
        if (along_r)
            k_line_pcr<true><<<dim3(blocks, nt), m, lds, s>>>(L.v, lam, u, f, color, mine);
        else
            k_line_pcr<false><<<dim3(blocks, nt), m, lds, s>>>(L.v, lam, u, f, color, mine);
        return hipGetLastError();
    }
    const dim3 grid((unsigned)((mine + 63) / 64), nt);
    if (along_r)
        k_rline<<<grid, 64, 0, s>>>(L.v, lam, u, f, scratch, color);
    else
        k_zline<<<grid, 64, 0, s>>>(L.v, lam, u, f, scratch, color);
    return hipGetLastError();
}

hipError_t launch_residual(const DeviceLevel& L, int nt, const double* lam, const double* u,
                           const double* f, double* r, hipStream_t s) {
    k_residual<<<grid_interior(L.v, nt), dim3(kTx, kTy), 0, s>>>(L.v, lam, u, f, r);
    return hipGetLastError();
}

hipError_t launch_restrict(const DeviceLevel& F, const DeviceLevel& C, int nt, const double* r,
                           double* fc, hipStream_t s) {
    k_restrict<<<grid_interior(C.v, nt), dim3(kTx, kTy), 0, s>>>(F.v, C.v, F.tr, F.tz, r, fc);
    return hipGetLastError();
}

hipError_t launch_prolong(const DeviceLevel& F, const DeviceLevel& C, int nt, const double* uc,
                          double* u, hipStream_t s, bool add) {
    if (add)
        k_prolong<true><<<grid_interior(F.v, nt), dim3(kTx, kTy), 0, s>>>(F.v, C.v, F.tr, F.tz, uc, u);
    else
        k_prolong<false><<<grid_interior(F.v, nt), dim3(kTx, kTy), 0, s>>>(F.v, C.v, F.tr, F.tz, uc, u);
    return hipGetLastError();
}

hipError_t launch_coarse_solve(const DeviceLevel& L, int nt, const double* lam, const double* cinv,
                               int n, const double* f, double* u, hipStream_t s) {
    k_coarse_solve<<<nt, 256, 2 * n * sizeof(double), s>>>(L.v, lam, cinv, n, f, u);
    return hipGetLastError();
}

hipError_t launch_init_ring(const DeviceLevel& L, int nt, const cylpoisson_bc& bc, hipStream_t s) {
    const int n = 2 * L.v.nr + 2 * (L.v.nz - 2);
    k_init_ring<<<dim3((n + 255) / 256, nt), 256, 0, s>>>(L.v, L.u, L.u2, bc.phi_r_in, bc.phi_r_out,
                                                          bc.phi_z0, bc.phi_zL);
    return hipGetLastError();
}


hipError_t launch_copy_ring(const DeviceLevel& L, int nt, const double* src, double* dst,
                            hipStream_t s) {
    const int n = 2 * L.v.nr + 2 * (L.v.nz - 2);
    k_copy_ring<<<dim3((n + 255) / 256, nt), 256, 0, s>>>(L.v, src, dst);
    return hipGetLastError();
}

}  // namespace cp
