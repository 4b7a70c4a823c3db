// Azimuthal transforms (Eq. azimuthal_dft) for any Ntheta up to 256 on the FP64
// matrix cores.  The dense N x N product is folded first: with
//   e_j = x_j + x_{N-j}, o_j = x_j - x_{N-j}   (0 < j < N/2; e_0 = x_0, e_{N/2} = x_{N/2})
// the planes are Re x^_m = sum_{j <= N/2} e_j cos(2 pi m j / N) / N and
// Im x^_m = -sum_{0 < j < N/2} o_j sin(2 pi m j / N) / N, two products of half
// the size each way; the inverse runs the same two products on the planes, E_j
// and O_j, and unfolds x_j = E_j + O_j, x_{N-j} = E_j - O_j.  A quarter of the
// dense product's operations in all, and each value of the input is read once.
//
// A wavefront takes 16 columns of the [Ntheta][Nz Nr] array by itself: every
// folded (or plane) value of its columns is loaded at once into registers, in
// the layout of the B operand (lane l holds rows 4 kb + l / 16, column l % 16),
// and each 16 x 16 tile of results is then two chains of
// v_mfma_f64_16x16x4f64 (lane l holds A[l % 16][l / 16], B[l / 16][l % 16] and
// D[l / 16 + 4 q][l % 16], q < 4).  The cosine and sine matrices are packed in
// the A operand's lane order when the plan is built, so an operand is one
// coalesced load, from L2 after the first wavefronts.
//
// What bounds it: at N = 96 the products need 9 us of the matrix cores for
// 51,200 columns and the columns' bytes 15 us at the rate of a large copy.
// Forward and inverse together took 56 us (271 us as dense
// products on the vector unit, whose matrix entries came one scalar load
// each; 90 us with 64 columns of a workgroup staged in LDS, whose load,
// product and store phases ran one after another in one wave of workgroups
// and a nearly empty second one).
#include "cp_internal.h"

#include <cmath>

namespace cp {

namespace {

typedef double dbl4 __attribute__((ext_vector_type(4)));

// KB: k-blocks of four azimuths (forward) or modes (inverse) held in registers.
template <bool INV, int KB>
__global__ void __launch_bounds__(256) k_dft_mfma(const double* __restrict__ Ac, const double* __restrict__ As,
                                                  const double* __restrict__ X, double* __restrict__ Y, int n, int kc,
                                                  long long ncols, const double* __restrict__ cs) {
    const int lane = threadIdx.x & 63, kr = lane >> 4;
    const long long col = ((long long)blockIdx.x * 4 + (threadIdx.x >> 6)) * 16 + (lane & 15);
    const bool in = col < ncols;
    const int half = n / 2, nc = half + 1, tiles = (nc + 15) / 16;
    const double* x = X + (in ? col : 0);
    double p[KB], q[KB];  // B operands of the cosine and the sine product
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        const int k = 4 * kb + kr;
        const bool pair = k > 0 && 2 * k < n;
        p[kb] = k < nc ? x[(long long)k * ncols] : 0.0;
        q[kb] = pair ? x[(long long)(INV ? half + k : n - k) * ncols] : 0.0;
    }
    if (!INV) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            const int k = 4 * kb + kr;
            const bool pair = k > 0 && 2 * k < n;
            const double a = p[kb], b = q[kb];
            p[kb] = a + b;
            q[kb] = pair ? a - b : 0.0;
        }
    }
    const double scale = !INV && cs && in ? cs[col] : 1.0;
    for (int tile = 0; tile < tiles; ++tile) {
        const double* ac = Ac + (long long)tile * kc * 64 + lane;
        const double* as = As + (long long)tile * kc * 64 + lane;
        dbl4 e = {0.0, 0.0, 0.0, 0.0}, o = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            const int b = KB > 17 ? min(kb, kc - 1) : kb;  // blocks past the last hold zero operands
            e = __builtin_amdgcn_mfma_f64_16x16x4f64(ac[b * 64], p[kb], e, 0, 0, 0);
            o = __builtin_amdgcn_mfma_f64_16x16x4f64(as[b * 64], q[kb], o, 0, 0, 0);
        }
        if (!in) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = 16 * tile + kr + 4 * r;
            if (m >= nc) continue;
            const bool pair = m > 0 && 2 * m < n;
            if (INV) {
                Y[(long long)m * ncols + col] = pair ? e[r] + o[r] : e[r];
                if (pair) Y[(long long)(n - m) * ncols + col] = e[r] - o[r];
            } else {
                Y[(long long)m * ncols + col] = e[r] * scale;
                if (pair) Y[(long long)(half + m) * ncols + col] = o[r] * scale;
            }
        }
    }
}

template <int KB>
hipError_t launch_kb(bool inv, int kc, const double* Ac, const double* As, const double* X, double* Y, int n,
                     long long ncols, const double* cs, hipStream_t s) {
    if constexpr (KB <= 17) {
        if (kc > KB) return launch_kb<KB + 1>(inv, kc, Ac, As, X, Y, n, ncols, cs, s);
    } else if constexpr (KB < 33) {
        if (kc > KB) return launch_kb<KB + 5>(inv, kc, Ac, As, X, Y, n, ncols, cs, s);
    }
    const unsigned blocks = (unsigned)((ncols + 63) / 64);
    if (inv)
        k_dft_mfma<true, KB><<<blocks, 256, 0, s>>>(Ac, As, X, Y, n, kc, ncols, cs);
    else
        k_dft_mfma<false, KB><<<blocks, 256, 0, s>>>(Ac, As, X, Y, n, kc, ncols, cs);
    return hipGetLastError();
}

}  // namespace

// Up to 256 azimuths: 33 k-blocks, 132 registers of operands.
bool dft_packed(int n) { return n <= 256; }

// The folded matrices in A operand order: forward cosine, forward sine,
// inverse cosine, inverse sine; off[i] is the first entry of matrix i.
void dft_pack(int n, std::vector<double>& out, size_t (&off)[4]) {
    const int nc = n / 2 + 1, kc = (nc + 3) / 4, tiles = (nc + 15) / 16;
    const double two_pi = 6.283185307179586476925286766559;
    out.clear();
    for (int i = 0; i < 4; ++i) {
        const bool inv = i >= 2, sine = i & 1;
        off[i] = out.size();
        for (int t = 0; t < tiles; ++t)
            for (int kb = 0; kb < kc; ++kb)
                for (int l = 0; l < 64; ++l) {
                    const int m = 16 * t + l % 16, k = 4 * kb + l / 16;
                    const bool pm = m > 0 && 2 * m < n, pk = k > 0 && 2 * k < n;
                    const double ang = two_pi * (double)(((long long)m * k) % n) / (double)n;
                    double v = 0.0;
                    if (sine) {
                        if (pm && pk) v = inv ? -2.0 * std::sin(ang) : -std::sin(ang) / (double)n;
                    } else if (m < nc && k < nc) {
                        // inverse: the weight of mode k, 1 for k = 0 and N/2
                        v = inv ? (pk ? 2.0 : 1.0) * std::cos(ang) : std::cos(ang) / (double)n;
                    }
                    out.push_back(v);
                }
    }
}

hipError_t launch_dft_packed(bool inverse, const double* A, const size_t (&off)[4], const double* X, double* Y, int n,
                             long long ncols, const double* cs, hipStream_t s) {
    const double* Ac = A + off[inverse ? 2 : 0];
    const double* As = A + off[inverse ? 3 : 1];
    return launch_kb<1>(inverse, (n / 2 + 4) / 4, Ac, As, X, Y, n, ncols, cs, s);
}

}  // namespace cp
