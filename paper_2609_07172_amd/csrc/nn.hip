// The learned preconditioner's network on the GPU: a three-layer 3x3
// convolution stack (4 -> 16 -> 16 -> 2 channels, ReLU after the first two,
// no biases) with BF16 operands and FP32 accumulation on the matrix cores
// (v_mfma_f32_16x16x16_bf16), for inference, back-propagation and training.
//
// Images are FP32 [B][H][W][C] (C fastest), zero outside the image.  Weights
// are FP32 masters [9][Cin][Cout] (tap t = (dy + 1) * 3 + (dx + 1)) with BF16
// copies packed in the lane order of a matrix-core operand, block kb of 16 by
// lane l: values k = 16 kb + 4 (l / 16) + j, j < 4, of column n = l % 16 of
//   forward   Wf[k = t * Cin + c][n = o]   (n padded to 16)
//   backward  Wb[k = t * Cout + o][n = c]
// A convolution is an implicit product over taps x input channels (K, in
// blocks of 16, the taps in order), output channels (M, 16) and pixels (N, 16
// of a row).  The weights are the first operand, so a lane holds four
// consecutive channels of one pixel of the result: one 8-byte LDS write.
// Operands are rounded from FP32 to BF16 (nearest, ties to even) as they are
// stored for a product, so an activation is rounded exactly where it enters one.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "cp_internal.h"
#include "nn_internal.h"

namespace cp {

namespace {

typedef short v4s __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

// images have the alignment of a float only
struct __attribute__((packed, aligned(4))) F4 {
    float v[4];
};
struct __attribute__((packed, aligned(4))) F2 {
    float v[2];
};

__device__ __forceinline__ short to_bf16(float x) {
    unsigned u = __float_as_uint(x);
    u = (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
    return (short)u;
}

// Four values at once (v_cvt_pk_bf16_f32: nearest, ties to even).
typedef __bf16 b2 __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ v4s to_bf16x4(float a, float b, float c, float d) {
    struct {
        b2 lo, hi;
    } r{__builtin_convertvector(f2{a, b}, b2), __builtin_convertvector(f2{c, d}, b2)};
    return __builtin_bit_cast(v4s, r);
}
// max(x, 0), 0 for NaN: a compare and a select (fmaxf quiets its operand first)
__device__ __forceinline__ float relu(float x) { return x > 0.f ? x : 0.f; }

// Orders the workgroup's LDS accesses only: global loads stay in flight.
__device__ __forceinline__ void lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ v4s operand(const short* __restrict__ wpk, int block, int lane) {
    return *(const v4s*)(wpk + ((size_t)block * 64 + lane) * 4);
}

// ---- forward: the three layers in one stream of rows ----
//
// A workgroup of NT wavefronts takes a strip of S = 16 NT pixels of an image
// (the outer three on each side recomputed by the neighbours) and marches
// down its rows; wavefront w computes pixels 16 w .. 16 w + 15 of every layer.
// At step k (row s = s0 + k) it forms row s of the first activation, row s - 2
// of the second and row s - 4 of the output, each from rows of earlier steps:
// one LDS-only barrier a step, and rings of 8, 4 and 2 rows in LDS.
//
// The last layer has two output channels: its products put (dy, o) on the
// result's rows instead, so that one input row takes three products (dx), and
// each output row's sum stays in its own lanes (row set R mod 3) while three
// input rows add their taps to it, in the order dy = -1, 0, 1.
//
// What bounds it: 15 products and 17 8-byte LDS accesses per 16 pixels and row
// keep the matrix cores and LDS about equally busy (95 us each for 13.2 million
// pixels), the image's bytes need 62 us.  Measured 185 us (388 us while an
// operand's lanes met on half the banks; 611 us in
// 16 x 32 tiles whose three layers ran between barriers, with a halo of three
// pixels on every side, index arithmetic per operand and nine products a row
// for the two output channels).
template <int NT, bool TRAIN>
struct Stream {
    static constexpr int S = 16 * NT, T = 64 * NT;
    // LDS rows (in shorts): an activation row holds its four groups of four
    // channels one after another, a pixel's 8 bytes next to its neighbours', and
    // a group's (an input row's) length is an odd multiple of 128 bytes, so that
    // an operand's lanes (16 pixels of four groups) cover every bank evenly
    static constexpr int kGroup = S == 32 ? 192 : 320;
    static constexpr int kInRow = kGroup;
    static constexpr int kActRow = 4 * kGroup;
    static_assert((S + 2) * 4 <= kGroup, "a row and the pixel past each end");
    static constexpr int kLds = 8 * kInRow + 6 * kActRow;

    const float* img;
    const float* timg;
    float *y, *a1g, *a2g;  // this image's output (gradient of the loss when TRAIN), activations
    short *in, *a1, *a2;
    int H, W, y0, y1, s0, margin;
    float inv_n;
    int t, lane, g, row, px, gx;
    bool colv, own;
    v4s w1[3], w2[9], w3[3][3];
    int in_dy[3], in_off[3];
    v4f out;       // sums of the output rows in flight
    F4 next;       // prefetched input pixel of this thread
    F2 tnext;      // prefetched target of the next output row
    double loss;

    __device__ __forceinline__ F4 fetch(int i) const {
        // input row index i (row s0 - 1 + i) of this thread's pixel
        const int r = s0 - 1 + i, c = gx - px + t % S;
        F4 v{{0.f, 0.f, 0.f, 0.f}};
        if (r >= 0 && r < H && c >= 0 && c < W) v = *(const F4*)(img + ((long long)r * W + c) * 4);
        return v;
    }
    __device__ __forceinline__ void put(int i, const F4& f) {
        *(v4s*)(in + (i & 7) * kInRow + (t % S + 1) * 4) = to_bf16x4(f.v[0], f.v[1], f.v[2], f.v[3]);
    }
    __device__ __forceinline__ F2 target(int R) const {
        F2 v{{0.f, 0.f}};
        if (TRAIN && own && R >= y0 && R < y1) v = *(const F2*)(timg + ((long long)R * W + gx) * 2);
        return v;
    }

    // An activation row's four channels of the lane's pixel: ReLU, zero
    // outside the image, BF16 to LDS; the FP32 values to memory for training.
    __device__ __forceinline__ void activation(v4f acc, int r, short* dst, float* __restrict__ gdst) {
        F4 f;
#pragma unroll
        for (int j = 0; j < 4; ++j) f.v[j] = relu(acc[j]);
        const v4s o = to_bf16x4(f.v[0], f.v[1], f.v[2], f.v[3]);
        const bool valid = colv && r >= 0 && r < H;
        *(v4s*)(dst + g * kGroup + (px + 1) * 4) = valid ? o : v4s{0, 0, 0, 0};
        if (TRAIN && own && r >= y0 && r < y1) *(F4*)(gdst + ((long long)r * W + gx) * 16 + 4 * g) = f;
    }

    template <int K>  // k mod 12
    __device__ __forceinline__ void step(int k) {
        lds_sync();
        const int s = s0 + k;
        if ((K & 3) == 1) {  // the batch of rows read from the next step on, and the loads of the one after
            put(k + 3 + t / S, next);
            next = fetch(k + 7 + t / S);
        }
        // every operand of the step is read first; the three layers' chains of
        // products then alternate
        v4s o1[3], o2[9], o3[3];
#pragma unroll
        for (int kb = 0; kb < 3; ++kb) o1[kb] = *(const v4s*)(in + ((k + 1 + in_dy[kb]) & 7) * kInRow + in_off[kb]);
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
            const int dy = tap / 3 - 1, dx = tap % 3 - 1;
            o2[tap] = *(const v4s*)(a1 + ((K - 2 + dy + 4) & 3) * kActRow + g * kGroup + (px + 1 + dx) * 4);
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) o3[d] = *(const v4s*)(a2 + ((K + 1) & 1) * kActRow + g * kGroup + (px + d) * 4);
        constexpr int v = K % 3;
        const bool fresh = g == (v + 1) % 3;
        out[0] = fresh ? 0.f : out[0];
        out[1] = fresh ? 0.f : out[1];
        v4f acc1 = {0.f, 0.f, 0.f, 0.f}, acc2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            acc1 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w1[d], o1[d], acc1, 0, 0, 0);
            acc2 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w2[d], o2[d], acc2, 0, 0, 0);
            out = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w3[v][d], o3[d], out, 0, 0, 0);
        }
#pragma unroll
        for (int tap = 3; tap < 9; ++tap) acc2 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w2[tap], o2[tap], acc2, 0, 0, 0);
        activation(acc1, s, a1 + (K & 3) * kActRow, a1g);
        activation(acc2, s - 2, a2 + (K & 1) * kActRow, a2g);
        const int R = s - 4;
        if (own && g == (v + 2) % 3 && R >= y0 && R < y1) {
            F2 o{{out[0], out[1]}};
            if (TRAIN) {
                const bool inner = R >= margin && R < H - margin && gx >= margin && gx < W - margin;
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const float d = inner ? o.v[c] - tnext.v[c] : 0.f;
                    o.v[c] = d * inv_n;
                    loss += (double)d * d;
                }
            }
            *(F2*)(y + ((long long)R * W + gx) * 2) = o;
        }
        if (TRAIN) tnext = target(R + 1);
    }

    template <int K>
    __device__ __forceinline__ void steps(int k0, int n) {
        if constexpr (K < 12) {
            if (k0 + K >= n) return;
            step<K>(k0 + K);
            steps<K + 1>(k0, n);
        }
    }

    __device__ __forceinline__ void run(const short* __restrict__ w0p, const short* __restrict__ w1p,
                                        const short* __restrict__ w2p, short* smem, int strip) {
        t = threadIdx.x;
        lane = t & 63;
        g = lane >> 4;
        row = lane & 15;
        px = 16 * (t >> 6) + row;
        gx = strip * (S - 6) - 3 + px;
        colv = gx >= 0 && gx < W;
        own = px >= 3 && px < S - 3 && gx < W;
        in = smem;
        a1 = in + 8 * kInRow;
        a2 = a1 + 4 * kActRow;
        s0 = y0 - 2;
        const F4 first = fetch(t / S);
        next = fetch(4 + t / S);
#pragma unroll
        for (int kb = 0; kb < 3; ++kb) {
            w1[kb] = operand(w0p, kb, lane);
            // block kb of the first layer holds taps 4 kb + g (four channels
            // each); past the ninth tap the weights are zero and the operand is
            // the zero before the row's first pixel (a pixel's own value may be
            // infinite)
            const int tap = min(4 * kb + g, 8);
            in_dy[kb] = tap / 3 - 1;
            in_off[kb] = 4 * kb + g <= 8 ? (px + 1 + tap % 3 - 1) * 4 : 0;
        }
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) w2[tap] = operand(w1p, tap, lane);
        // version v of the last layer: rows 4 q + o take tap dy of (q - v) mod 3
        const int q = row >> 2, o = row & 3;
#pragma unroll
        for (int v = 0; v < 3; ++v)
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const int rel = (q - v + 3) % 3;  // 1: first (dy = -1), 0: second, 2: last
                const int tap = (rel == 1 ? 0 : rel == 0 ? 3 : 6) + d;
                const v4s w = operand(w2p, tap, 16 * g + (o & 1));
#pragma unroll
                for (int j = 0; j < 4; ++j) w3[v][d][j] = q < 3 && o < 2 ? w[j] : (short)0;
            }
        out = v4f{0.f, 0.f, 0.f, 0.f};
        loss = 0.0;
        tnext = F2{{0.f, 0.f}};
        // rows of earlier steps read before the first ones are formed, and the
        // pixel past each end of a row: zero
        for (int i = t; i < kLds; i += T) smem[i] = 0;
        lds_sync();
        put(t / S, first);
        const int n = y1 - y0 + 6;
        for (int k0 = 0; k0 < n; k0 += 12) steps<0>(k0, n);
    }
};

template <int NT, bool TRAIN>
__global__ void __launch_bounds__(64 * NT, 4) k_net(const float* __restrict__ x, const short* __restrict__ w0,
                                                 const short* __restrict__ w1, const short* __restrict__ w2,
                                                 float* __restrict__ y, const float* __restrict__ target,
                                                 float* __restrict__ a1, float* __restrict__ a2,
                                                 double* __restrict__ partial, int H, int W, int rows, int strips, int chunks,
                                                 int margin, float inv_n) {
    __shared__ __attribute__((aligned(16))) short smem[Stream<NT, TRAIN>::kLds];
    Stream<NT, TRAIN> st;
    const int per = strips * chunks, q = (int)(blockIdx.x % per);
    const long long pix = (long long)(blockIdx.x / per) * H * W;
    st.img = x + pix * 4;
    st.y = y + pix * 2;
    st.timg = TRAIN ? target + pix * 2 : nullptr;
    st.a1g = TRAIN ? a1 + pix * 16 : nullptr;
    st.a2g = TRAIN ? a2 + pix * 16 : nullptr;
    st.H = H;
    st.W = W;
    st.y0 = (q / strips) * rows;
    st.y1 = min(H, st.y0 + rows);
    st.margin = margin;
    st.inv_n = inv_n;
    st.run(w0, w1, w2, smem, q % strips);
    if (TRAIN) {
        // fixed-order sum of the squared differences over the workgroup
        double s = st.loss;
#pragma unroll
        for (int w = 32; w > 0; w >>= 1) s += __shfl_xor(s, w);
        __syncthreads();
        double* red = (double*)smem;
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
        __syncthreads();
        if (threadIdx.x == 0) {
            double a = 0.0;
            for (int i = 0; i < NT; ++i) a += red[i];
            partial[blockIdx.x] = a;
        }
    }
}

// ---- backward: both data gradients and the three weight gradients ----
//
// A workgroup takes 16 x 32 pixel tiles, one after another: the tile's
// activations, input (halo 1) and output gradient (halo 2) go to LDS as BF16,
// then g2 = conv^T(g3) where a2 > 0 (halo 1), g1 = conv^T(g2) where a1 > 0, and
// each weight gradient dW[t, c][o] = sum_p act[p + off_t][c] g[p][o] as a
// product with 16 pixels of a row as K, accumulated in registers over the
// workgroup's tiles; the wavefronts' sums are added in LDS and written as one
// partial per workgroup (added up in a fixed order by k_reduce).
//
// What bounds it: latency, at one workgroup per compute unit.  A training step
// on 128 patches of 32 x 32 takes 20 us forward, 17 us here and 8 us for the
// sums and Adam (90 us with the read-backs of loss, gradients and weights);
// one kernel per layer, and sums over 512 partials by one thread per weight
// (3 x 125 us), took 615 us.
constexpr int kBH = 16, kBW = 32;                  // tile: rows x columns
constexpr int kP = 20;                             // LDS shorts per pixel of 16 channels (bank spread)
constexpr int kHalo1 = (kBH + 2) * (kBW + 2), kHalo2 = (kBH + 4) * (kBW + 4);
constexpr int kBThreads = 512, kBWaves = kBThreads / 64;
constexpr int kPart1 = 3 * 256, kPart2 = 9 * 256, kPart = kPart1 + 2 * kPart2;  // dW1, dW2, dW3 rows of 16
constexpr int kBLds = 3 * kHalo1 * kP + kBH * kBW * kP + kHalo2 * 2 + kHalo1 * 4;  // shorts
static_assert(kBLds * 2 >= kBWaves * kPart2 * 4, "the partial sums fit where the tile was");

__global__ void __launch_bounds__(kBThreads) k_net_bwd(const float* __restrict__ x, const float* __restrict__ a1,
                                                       const float* __restrict__ a2, const float* __restrict__ g3,
                                                       const short* __restrict__ wb1, const short* __restrict__ wb2,
                                                       float* __restrict__ partial, int H, int W, int tiles_x,
                                                       int tiles_y, int ntiles) {
    extern __shared__ __attribute__((aligned(16))) short smb[];
    short* A1 = smb;
    short* A2 = A1 + kHalo1 * kP;
    short* G2 = A2 + kHalo1 * kP;
    short* G1 = G2 + kHalo1 * kP;
    short* G3 = G1 + kBH * kBW * kP;
    short* X = G3 + kHalo2 * 2;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, g = lane >> 4, row = lane & 15;
    v4f acc1[3], acc2[9], acc3[9];
#pragma unroll
    for (int m = 0; m < 9; ++m) {
        if (m < 3) acc1[m] = v4f{0.f, 0.f, 0.f, 0.f};
        acc2[m] = acc3[m] = v4f{0.f, 0.f, 0.f, 0.f};
    }
    v4s w2[2], w1[9];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) w2[kb] = operand(wb2, kb, lane);
#pragma unroll
    for (int kb = 0; kb < 9; ++kb) w1[kb] = operand(wb1, kb, lane);
    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int b = tile / (tiles_x * tiles_y), q = tile % (tiles_x * tiles_y);
        const int y0 = (q / tiles_x) * kBH, x0 = (q % tiles_x) * kBW;
        const long long pix = (long long)b * H * W;
        // four channels of a halo pixel per item
        constexpr int NA = (kHalo1 * 4 + kBThreads - 1) / kBThreads, NX = (kHalo1 + kBThreads - 1) / kBThreads,
                      NG = (kHalo2 + kBThreads - 1) / kBThreads;
        F4 la[2][NA], lx[NX];
        F2 lg[NG];
#pragma unroll
        for (int u = 0; u < NA; ++u) {
            const int i = t + u * kBThreads, p = i >> 2, c = (i & 3) * 4;
            const int yy = y0 - 1 + p / (kBW + 2), xx = x0 - 1 + p % (kBW + 2);
            const bool in = i < kHalo1 * 4 && yy >= 0 && yy < H && xx >= 0 && xx < W;
            const long long o = (pix + (long long)yy * W + xx) * 16 + c;
            la[0][u] = la[1][u] = F4{{0.f, 0.f, 0.f, 0.f}};
            if (in) {
                la[0][u] = *(const F4*)(a1 + o);
                la[1][u] = *(const F4*)(a2 + o);
            }
        }
#pragma unroll
        for (int u = 0; u < NX; ++u) {
            const int p = t + u * kBThreads;
            const int yy = y0 - 1 + p / (kBW + 2), xx = x0 - 1 + p % (kBW + 2);
            lx[u] = F4{{0.f, 0.f, 0.f, 0.f}};
            if (p < kHalo1 && yy >= 0 && yy < H && xx >= 0 && xx < W)
                lx[u] = *(const F4*)(x + (pix + (long long)yy * W + xx) * 4);
        }
#pragma unroll
        for (int u = 0; u < NG; ++u) {
            const int p = t + u * kBThreads;
            const int yy = y0 - 2 + p / (kBW + 4), xx = x0 - 2 + p % (kBW + 4);
            lg[u] = F2{{0.f, 0.f}};
            if (p < kHalo2 && yy >= 0 && yy < H && xx >= 0 && xx < W)
                lg[u] = *(const F2*)(g3 + (pix + (long long)yy * W + xx) * 2);
        }
        __syncthreads();  // the previous tile's last reads
#pragma unroll
        for (int u = 0; u < NA; ++u) {
            const int i = t + u * kBThreads, p = i >> 2, c = (i & 3) * 4;
            if (i >= kHalo1 * 4) continue;
            v4s o1, o2;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                o1[j] = to_bf16(la[0][u].v[j]);
                o2[j] = to_bf16(la[1][u].v[j]);
            }
            *(v4s*)(A1 + p * kP + c) = o1;
            *(v4s*)(A2 + p * kP + c) = o2;
        }
#pragma unroll
        for (int u = 0; u < NX; ++u) {
            const int p = t + u * kBThreads;
            if (p >= kHalo1) continue;
            v4s o;
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j] = to_bf16(lx[u].v[j]);
            *(v4s*)(X + p * 4) = o;
        }
#pragma unroll
        for (int u = 0; u < NG; ++u) {
            const int p = t + u * kBThreads;
            if (p >= kHalo2) continue;
            G3[2 * p] = to_bf16(lg[u].v[0]);
            G3[2 * p + 1] = to_bf16(lg[u].v[1]);
        }
        __syncthreads();
        // g2 on the tile and its halo: K = (tap, output channel), two taps of a lane's four values
        for (int q2 = wave; q2 < (kHalo1 + 15) / 16; q2 += kBWaves) {
            const int p = q2 * 16 + row;
            const int pr = min(p, kHalo1 - 1) / (kBW + 2), pc = min(p, kHalo1 - 1) % (kBW + 2);
            v4f acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                v4s bv;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    // past the ninth tap the weights are zero, and so is the
                    // operand (a gradient may be infinite)
                    const int k = kb * 8 + 2 * g + h, tap = min(k, 8);
                    const short* s = G3 + ((pr + 1 - (tap / 3 - 1)) * (kBW + 4) + pc + 1 - (tap % 3 - 1)) * 2;
                    bv[2 * h] = k <= 8 ? s[0] : (short)0;
                    bv[2 * h + 1] = k <= 8 ? s[1] : (short)0;
                }
                acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w2[kb], bv, acc, 0, 0, 0);
            }
            if (p < kHalo1) {
                const int yy = y0 - 1 + pr, xx = x0 - 1 + pc;
                const bool in = yy >= 0 && yy < H && xx >= 0 && xx < W;
                const v4s m = *(const v4s*)(A2 + p * kP + 4 * g);
                v4s o;
#pragma unroll
                for (int j = 0; j < 4; ++j) o[j] = in && m[j] > 0 ? to_bf16(acc[j]) : (short)0;
                *(v4s*)(G2 + p * kP + 4 * g) = o;
            }
        }
        __syncthreads();
        // g1 on the tile
        for (int q1 = wave; q1 < kBH * kBW / 16; q1 += kBWaves) {
            const int pr = q1 / (kBW / 16), pc = (q1 % (kBW / 16)) * 16 + row;
            v4f acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int tap = 0; tap < 9; ++tap) {
                const int dy = tap / 3 - 1, dx = tap % 3 - 1;
                acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
                    w1[tap], *(const v4s*)(G2 + ((pr + 1 - dy) * (kBW + 2) + pc + 1 - dx) * kP + 4 * g), acc, 0, 0, 0);
            }
            const bool in = y0 + pr < H && x0 + pc < W;
            const v4s m = *(const v4s*)(A1 + ((pr + 1) * (kBW + 2) + pc + 1) * kP + 4 * g);
            v4s o;
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j] = in && m[j] > 0 ? to_bf16(acc[j]) : (short)0;
            *(v4s*)(G1 + (pr * kBW + pc) * kP + 4 * g) = o;
        }
        __syncthreads();
        // weight gradients: blocks of 16 pixels of a row, lane l holds pixels
        // 4 (l / 16) + j of channel (or weight row) l % 16
#pragma unroll 1
        for (int blk = wave; blk < kBH * kBW / 16; blk += kBWaves) {
            const int pr = blk / (kBW / 16), pc = (blk % (kBW / 16)) * 16 + 4 * g;
            // a pixel outside the image has a zero gradient and must have a zero
            // activation too: the one beside it may be infinite
            if (y0 + pr >= H) continue;
            v4s in;  // all ones for those of the lane's four pixels in the image
#pragma unroll
            for (int j = 0; j < 4; ++j) in[j] = x0 + pc + j < W ? (short)-1 : (short)0;
            v4s b1, b2, b3;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                b1[j] = G1[(pr * kBW + pc + j) * kP + row];
                b2[j] = G2[((pr + 1) * (kBW + 2) + pc + 1 + j) * kP + row];
                b3[j] = row < 2 ? G3[((pr + 2) * (kBW + 4) + pc + 2 + j) * 2 + row] : (short)0;
            }
#pragma unroll
            for (int dy = 0; dy < 3; ++dy) {
                short e1[6], e2[6];
#pragma unroll
                for (int j = 0; j < 6; ++j) {
                    const int o = ((pr + dy) * (kBW + 2) + pc + j) * kP + row;
                    e1[j] = A1[o];
                    e2[j] = A2[o];
                }
#pragma unroll
                for (int dx = 0; dx < 3; ++dx) {
                    const v4s c1 = v4s{e1[dx], e1[dx + 1], e1[dx + 2], e1[dx + 3]} & in;
                    const v4s c2 = v4s{e2[dx], e2[dx + 1], e2[dx + 2], e2[dx + 3]} & in;
                    acc2[3 * dy + dx] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(c1, b2, acc2[3 * dy + dx], 0, 0, 0);
                    acc3[3 * dy + dx] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(c2, b3, acc3[3 * dy + dx], 0, 0, 0);
                }
            }
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                const int r = m * 16 + row, tap = min(r >> 2, 8);
                v4s c;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const short v = X[((pr + tap / 3) * (kBW + 2) + pc + tap % 3 + j) * 4 + (r & 3)];
                    c[j] = r < 36 ? v : (short)0;
                }
                c &= in;
                acc1[m] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(c, b1, acc1[m], 0, 0, 0);
            }
        }
    }
    // acc[m][j] = row 16 m + 4 g + j, column `row`
    float* red = (float*)smb;
    float* out = partial + (long long)blockIdx.x * kPart;
    auto reduce = [&](const v4f* acc, int tiles, float* dst) {
        __syncthreads();
#pragma unroll
        for (int m = 0; m < 9; ++m)
            if (m < tiles)
#pragma unroll
                for (int j = 0; j < 4; ++j) red[wave * tiles * 256 + (m * 16 + g * 4 + j) * 16 + row] = acc[m][j];
        __syncthreads();
        for (int i = t; i < tiles * 256; i += kBThreads) {
            float s = 0.f;
#pragma unroll
            for (int w = 0; w < kBWaves; ++w) s += red[w * tiles * 256 + i];
            dst[i] = s;
        }
    };
    v4f a1x[9];
#pragma unroll
    for (int m = 0; m < 9; ++m) a1x[m] = m < 3 ? acc1[m] : v4f{0.f, 0.f, 0.f, 0.f};
    reduce(a1x, 3, out);
    reduce(acc2, 9, out + kPart1);
    reduce(acc3, 9, out + kPart1 + kPart2);
}

// dw = the sum of the workgroups' partials (16 values a block, 16 slices of
// the partials each, added in a fixed order), and in the last block the loss
// sum of the forward's partials.
__global__ void __launch_bounds__(256) k_reduce(const float* __restrict__ partial, int nparts, float* __restrict__ dw,
                                                const double* __restrict__ loss, int nloss, double* __restrict__ loss_out) {
    const int t = threadIdx.x;
    if (blockIdx.x == kPart / 16) {
        __shared__ double redd[256];
        double s = 0.0;
        for (int i = t; i < nloss; i += 256) s += loss[i];
        redd[t] = s;
        __syncthreads();
        for (int w = 128; w > 0; w >>= 1) {
            if (t < w) redd[t] += redd[t + w];
            __syncthreads();
        }
        if (t == 0) *loss_out = redd[0];
        return;
    }
    __shared__ float red[16][17];
    const int o = t & 15, slice = t >> 4, q = blockIdx.x * 16 + o;
    float s = 0.f;
#pragma unroll 8
    for (int i = slice; i < nparts; i += 16) s += partial[(long long)i * kPart + q];
    red[slice][o] = s;
    __syncthreads();
    if (t >= 16) return;
    s = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) s += red[i][t];
    // weight row r = t * Cin + c and output channel o of its layer
    const int layer = q < kPart1 ? 0 : q < kPart1 + kPart2 ? 1 : 2;
    const int r = (q - (layer == 0 ? 0 : layer == 1 ? kPart1 : kPart1 + kPart2)) >> 4;
    const int cin = layer == 0 ? 4 : 16, cout = layer == 2 ? 2 : 16;
    const int off = layer == 0 ? 0 : layer == 1 ? 9 * 4 * 16 : 9 * 4 * 16 + 9 * 16 * 16;
    if (r < 9 * cin && t < cout) dw[off + r * cout + t] = s;
}

struct Packs {
    short *wf[3], *wb[3];
};

// Position of (k, n) in an operand pack.
__host__ __device__ inline int pack_at(int k, int n) { return ((k >> 4) * 64 + ((k >> 2) & 3) * 16 + n) * 4 + (k & 3); }

// Adam on the FP32 masters of all layers (flattened) and their BF16 packs.
__global__ void k_adam(float* __restrict__ w, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, Packs pk, int n, float lr, float b1, float b2, float eps, float c1,
                       float c2) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    const float gq = g[q];
    const float mq = b1 * m[q] + (1.f - b1) * gq;
    const float vq = b2 * v[q] + (1.f - b2) * gq * gq;
    m[q] = mq;
    v[q] = vq;
    const float wq = w[q] - lr * (mq / c1) / (sqrtf(vq / c2) + eps);
    w[q] = wq;
    const int l = q < 576 ? 0 : q < 2880 ? 1 : 2;
    const int cin = l == 0 ? 4 : 16, cout = l == 2 ? 2 : 16;
    const int r = q - (l == 0 ? 0 : l == 1 ? 576 : 2880);
    const int o = r % cout, c = (r / cout) % cin, t = r / (cout * cin);
    const short s = to_bf16(wq);
    pk.wf[l][pack_at(t * cin + c, o)] = s;
    pk.wb[l][pack_at(t * cout + o, c)] = s;
}

// The packs of one layer, padding included.
__global__ void k_pack(const float* __restrict__ w, short* __restrict__ wf, short* __restrict__ wb, int cin,
                       int cout) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;  // over KPf * 16 and KPb * 16
    const int kpf = (9 * cin + 15) / 16 * 16, kpb = (9 * cout + 15) / 16 * 16;
    const int k = q / 16, n = q % 16;
    if (k < kpf) {
        float v = 0.f;
        if (k < 9 * cin && n < cout) v = w[k * cout + n];
        wf[pack_at(k, n)] = to_bf16(v);
    }
    if (k < kpb) {
        float v = 0.f;
        if (k < 9 * cout && n < cin) v = w[((k / cout) * cin + n) * cout + k % cout];  // k = t * cout + o, n = c
        wb[pack_at(k, n)] = to_bf16(v);
    }
}

const int kCin[3] = {4, 16, 16};
const int kCout[3] = {16, 16, 2};

// Launch shape of the forward stream: wavefronts of a strip, strips of a row
// and rows of a chunk.  A strip of S pixels yields S - 6; images too narrow for
// 48 take one or two wavefronts fewer.  The chunks are as few as give about
// 1024 workgroups (four a compute unit), each recomputing six rows.
struct NetShape {
    int nt, strips, rows, chunks;
};
NetShape net_shape(int B, int H, int W) {
    NetShape s;
    s.nt = W <= 26 ? 2 : W <= 42 ? 3 : 4;
    s.strips = (W + 16 * s.nt - 7) / (16 * s.nt - 6);
    const long long per = (long long)B * s.strips;
    const int want = (int)std::max<long long>(1, kNetWgs / std::max<long long>(1, per));
    s.rows = std::max(8, (H + want - 1) / want);
    s.chunks = (H + s.rows - 1) / s.rows;
    return s;
}

template <bool TRAIN>
hipError_t launch_net(const NetShape& sh, NetState* n, const float* x, float* y, const float* t, int B, int H, int W,
                      float inv_n, hipStream_t s) {
    const long long blocks = (long long)sh.strips * sh.chunks * B;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    const unsigned grid = (unsigned)blocks;
    const int m = kNetMargin;
#define CP_NET(NT)                                                                                              \
    k_net<NT, TRAIN><<<grid, 64 * NT, 0, s>>>(x, n->wf[0], n->wf[1], n->wf[2], y, t, n->a1, n->a2, n->loss_partial, \
                                              H, W, sh.rows, sh.strips, sh.chunks, m, inv_n)
    if (sh.nt == 2)
        CP_NET(2);
    else if (sh.nt == 3)
        CP_NET(3);
    else
        CP_NET(4);
#undef CP_NET
    return hipGetLastError();
}

}  // namespace

size_t net_weight_offset(int l) {
    size_t o = 0;
    for (int i = 0; i < l; ++i) o += (size_t)9 * kCin[i] * kCout[i];
    return o;
}

hipError_t net_repack(NetState* n, hipStream_t s) {
    for (int l = 0; l < 3; ++l) {
        const int q = std::max((9 * kCin[l] + 15) / 16 * 16, (9 * kCout[l] + 15) / 16 * 16) * 16;
        k_pack<<<(q + 255) / 256, 256, 0, s>>>(n->w + net_weight_offset(l), n->wf[l], n->wb[l], kCin[l],
                                               kCout[l]);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

size_t net_partial_floats() { return (size_t)kNetPartials * kPart; }

namespace {

// Room for the activations and output gradient of `pixels` pixels and `sums` loss sums.
hipError_t net_reserve(NetState* n, long long pixels, long long sums) {
    if (pixels > n->capacity) {
        for (float* p : {n->a1, n->a2, n->g3})
            if (p) (void)hipFree(p);
        n->a1 = n->a2 = n->g3 = nullptr;
        n->capacity = 0;
        hipError_t e = hipMalloc(&n->a1, pixels * 16 * sizeof(float));
        if (e == hipSuccess) e = hipMalloc(&n->a2, pixels * 16 * sizeof(float));
        if (e == hipSuccess) e = hipMalloc(&n->g3, pixels * 2 * sizeof(float));
        if (e != hipSuccess) return e;
        n->capacity = pixels;
    }
    if (sums > n->loss_capacity) {
        if (n->loss_partial) (void)hipFree(n->loss_partial);
        n->loss_partial = nullptr;
        n->loss_capacity = 0;
        const hipError_t e = hipMalloc(&n->loss_partial, (sums + 1) * sizeof(double));  // the last: their sum
        if (e != hipSuccess) return e;
        n->loss_capacity = sums;
    }
    return hipSuccess;
}

}  // namespace

hipError_t net_infer(NetState* n, const float* x, float* y, int B, int H, int W, hipStream_t s) {
    if (B <= 0 || H <= 0 || W <= 0) return hipSuccess;
    return launch_net<false>(net_shape(B, H, W), n, x, y, nullptr, B, H, W, 0.f, s);
}

hipError_t net_loss_grad(NetState* n, const float* x, const float* t, int B, int H, int W, double* loss,
                         hipStream_t s) {
    const NetShape sh = net_shape(B, H, W);
    const long long sums = (long long)B * sh.strips * sh.chunks;
    hipError_t e = net_reserve(n, (long long)B * H * W, sums);
    if (e != hipSuccess) return e;
    const int m = kNetMargin;
    const long long inner = (long long)B * std::max(0, H - 2 * m) * std::max(0, W - 2 * m) * 2;
    const float inv_n = inner > 0 ? 1.f / (float)inner : 0.f;
    e = launch_net<true>(sh, n, x, n->g3, t, B, H, W, inv_n, s);
    if (e != hipSuccess) return e;
    const int tx = (W + kBW - 1) / kBW, ty = (H + kBH - 1) / kBH;
    const long long ntiles = (long long)B * tx * ty;
    if (ntiles > 0x7fffffff) return hipErrorInvalidValue;
    const int wgs = (int)std::min<long long>(kNetPartials, ntiles);
    // more than the default 64 KB of dynamic LDS: allowed on the current device
    // at every launch (a host call of a few microseconds)
    e = hipFuncSetAttribute((const void*)k_net_bwd, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(kBLds * sizeof(short)));
    if (e != hipSuccess) return e;
    k_net_bwd<<<wgs, kBThreads, kBLds * sizeof(short), s>>>(x, n->a1, n->a2, n->g3, n->wb[1], n->wb[2], n->partial, H,
                                                            W, tx, ty, (int)ntiles);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    double* sum = n->loss_partial + n->loss_capacity;
    k_reduce<<<kPart / 16 + 1, 256, 0, s>>>(n->partial, wgs, n->dw, n->loss_partial, (int)sums, sum);
    e = hipGetLastError();
    if (e == hipSuccess && loss) {
        e = hipMemcpyAsync(n->h_loss, sum, sizeof(double), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) return e;
        *loss = inner > 0 ? *n->h_loss / (2.0 * (double)inner) : 0.0;
    }
    return e;
}

hipError_t net_adam(NetState* n, float lr, hipStream_t s) {
    n->step += 1;
    const float b1 = 0.9f, b2 = 0.999f;
    const float c1 = 1.f - std::pow(b1, (float)n->step), c2 = 1.f - std::pow(b2, (float)n->step);
    const int total = (int)net_weight_offset(3);
    const Packs pk{{n->wf[0], n->wf[1], n->wf[2]}, {n->wb[0], n->wb[1], n->wb[2]}};
    k_adam<<<(total + 255) / 256, 256, 0, s>>>(n->w, n->dw, n->m, n->v, pk, total, lr, b1, b2, 1e-8f, c1, c2);
    return hipGetLastError();
}

int net_total_weights() { return (int)net_weight_offset(3); }

}  // namespace cp
