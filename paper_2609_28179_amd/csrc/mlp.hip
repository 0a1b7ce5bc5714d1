// mlp.hip -- training and inference kernels of the placement cost model, a
// 3-layer perceptron d -> 64 -> 64 -> 1 (ReLU) that predicts the log run time
// of a placement from (op, n, batch, scope, pack) features.  The paper picks
// placements by measurement only (Sec. III-A, Sec. IV-A); this model proposes
// placements for shapes that were not measured, with measured search as the
// fallback and as what decides among its picks.
//
// Parameter vector (flat): W1 [64][d], b1 [64], W2 [64][64], b2 [64],
// w3 [64], b3 [1].  A workgroup of four wavefronts works on a tile of
// samples, wavefront w owning hidden units 16 w .. 16 w + 15, and every
// product over units or samples runs on the matrix cores
// (v_mfma_f32_16x16x4_f32, FP32 throughout).  The backward pass writes
// per-block partial gradients that a second kernel sums over blocks in a
// fixed order, so training is deterministic (no floating-point atomics).
//
// Operand layouts (lane (q, r) = (lane / 16, lane % 16), element c of four):
// the left operand M holds M[r][4 q + c], the right operand X holds
// X[4 q + c][r], and D = M X comes out as D[4 q + c][r], so a product's result
// is the next one's right operand as it stands.
#include "device_common.hpp"
#include "glass_internal.hpp"

namespace glass {
namespace {

constexpr int kH = 64;
constexpr int kFwdSamples = 16;   // samples of a forward workgroup: one tile
constexpr int kBwdSamples = 32;   // samples of a backward tile (two 16-sample halves)
constexpr int kBwdBlocks = 256;   // most backward workgroups: one per compute unit
constexpr int kRedParams = 64, kRedSegs = 16;  // parameters and segments of a reduction workgroup

typedef float f4m_t __attribute__((ext_vector_type(4)));

GLASS_DEV f4m_t mlp_mma(const f4m_t& m, const f4m_t& x, f4m_t c) {
#pragma unroll
    for (int s = 0; s < 4; ++s) c = __builtin_amdgcn_mfma_f32_16x16x4f32(m[s], x[s], c, 0, 0, 0);
    return c;
}

// v summed over the four 16-lane rows of the wavefront, in every lane.
GLASS_DEV float sum_q(float v) {
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    return v;
}

// Element [row][col .. col + 3] of a row-major matrix of row length d, zero
// past the row's end; every load is unconditional (the row's first element
// instead), so that all of a tile's loads are in flight together.
GLASS_DEV f4m_t row_piece(const float* __restrict__ M, size_t row, int d, int col) {
    f4m_t v;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const float x = M[row * d + (col + c < d ? col + c : 0)];
        v[c] = col + c < d ? x : 0.f;
    }
    return v;
}

struct Off {
    int W1, b1, W2, b2, w3, b3, total;
};

__host__ __device__ inline Off offsets(int d) {
    Off o;
    o.W1 = 0;
    o.b1 = kH * d;
    o.W2 = o.b1 + kH;
    o.b2 = o.W2 + kH * kH;
    o.w3 = o.b2 + kH;
    o.b3 = o.w3 + kH;
    o.total = o.b3 + 1;
    return o;
}

// Sixteen samples per workgroup.  H1 = relu(W1 X^T + b1) tile by tile, the
// four tiles exchanged through LDS in operand layout (16 bytes a lane, no
// conflicts), then H2 and its product with w3.  Launch-bound: the weights
// are 21 KB read from L2 by every workgroup, and a wavefront issues 8 + 16
// MFMA.  One wavefront per 16 samples with a lane per hidden unit ran the
// samples one after the other through LDS broadcasts: at 4170 samples, d = 15,
// 16.9 us against 4.8 us now.
__global__ void __launch_bounds__(256) mlp_forward_k(int N, int d, const float* __restrict__ X,
                                                      const float* __restrict__ P, float* __restrict__ H1,
                                                      float* __restrict__ H2, float* __restrict__ Y) {
    __shared__ f4m_t h1s[4][64];
    __shared__ float ys[4][kFwdSamples];
    const int w = wave_index(), lane = threadIdx.x & 63, q = lane >> 4, r = lane & 15;
    const Off o = offsets(d);
    const int s = blockIdx.x * kFwdSamples + r;  // this lane's sample (column r of every tile)
    const bool in = s < N;
    const size_t sl = in ? s : N - 1;
    const int unit = 16 * w + 4 * q;             // this lane's four hidden units of a result
    f4m_t w1[2], x[2], w2[4], b1, b2, w3;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
        w1[kb] = row_piece(P + o.W1, 16 * w + r, d, 16 * kb + 4 * q);
        x[kb] = row_piece(X, sl, d, 16 * kb + 4 * q);
    }
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) w2[kb] = row_piece(P + o.W2, 16 * w + r, kH, 16 * kb + 4 * q);
    b1 = row_piece(P + o.b1, 0, kH, unit);
    b2 = row_piece(P + o.b2, 0, kH, unit);
    w3 = row_piece(P + o.w3, 0, kH, unit);
    const float b3 = P[o.b3];
    f4m_t h = mlp_mma(w1[0], x[0], b1);
    if (d > 16) h = mlp_mma(w1[1], x[1], h);
#pragma unroll
    for (int c = 0; c < 4; ++c) h[c] = fmaxf(h[c], 0.f);
    h1s[w][lane] = h;
    if (H1 && in) {
#pragma unroll
        for (int c = 0; c < 4; ++c) H1[sl * kH + unit + c] = h[c];
    }
    __syncthreads();
    f4m_t g = b2;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) g = mlp_mma(w2[kb], h1s[kb][lane], g);
    float y = 0.f;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        g[c] = fmaxf(g[c], 0.f);
        y = fmaf(w3[c], g[c], y);
    }
    if (H2 && in) {
#pragma unroll
        for (int c = 0; c < 4; ++c) H2[sl * kH + unit + c] = g[c];
    }
    y = sum_q(y);
    if (q == 0) ys[w][r] = y;
    __syncthreads();
    if (w == 0 && q == 0 && in) Y[s] = ((ys[0][r] + ys[1][r]) + (ys[2][r] + ys[3][r])) + b3;
}

// Partial gradients of L = (1/N) sum (y - t)^2 over this workgroup's tiles of
// 32 samples (tiles blockIdx.x, blockIdx.x + gridDim.x, ...):
//   gW2   = dH2^T H1            M = dH2^T (this wavefront's units), X = H1
//   dH1   = (dH2 W2) * [H1 > 0] M = dH2 (all units), X = W2
//   gW1^T = X^T dH1             M = X^T, X = dH1 as it comes out
// with dH2 = [H2 > 0] dy w3^T formed in either layout from H2 as loaded.
// Samples past N are cleared.  Bound by one round of loads and 80 dependent-
// free MFMA per wavefront and tile; a lane per hidden unit with the samples
// one after the other took 36.2 us at 4170 samples, d = 15, against 8.0 us now.
// At most kBwdBlocks partial vectors are written: they are what the
// reduction reads back.
__global__ void __launch_bounds__(256) mlp_backward_k(int N, int d, const float* __restrict__ X,
                                                       const float* __restrict__ P, const float* __restrict__ H1,
                                                       const float* __restrict__ H2, const float* __restrict__ Y,
                                                       const float* __restrict__ T, float* __restrict__ part) {
    const int w = wave_index(), lane = threadIdx.x & 63, q = lane >> 4, r = lane & 15;
    const Off o = offsets(d);
    const int unit = 16 * w + r;  // this lane's hidden unit (column r of the wavefront's tiles)
    f4m_t w2[4], w3t[4];
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) {
#pragma unroll
        for (int c = 0; c < 4; ++c) w2[jb][c] = P[o.W2 + (16 * jb + 4 * q + c) * kH + unit];
        w3t[jb] = row_piece(P + o.w3, 0, kH, 16 * jb + 4 * q);
    }
    const float w3 = P[o.w3 + unit];
    const f4m_t zero = {0.f, 0.f, 0.f, 0.f};
    f4m_t gW2[4] = {zero, zero, zero, zero}, gW1[2] = {zero, zero};
    float gb1 = 0.f, gb2 = 0.f, gw3 = 0.f, gb3 = 0.f;
    const float scale = 2.0f / (float)N;
    for (long long t0 = (long long)blockIdx.x * kBwdSamples; t0 < N; t0 += (long long)gridDim.x * kBwdSamples) {
        f4m_t h1[2][4], h2t[2][4], h2[2], dy[2], xt[2][2];
        float dyr[2];
#pragma unroll
        for (int sb = 0; sb < 2; ++sb) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const long long s = t0 + 16 * sb + 4 * q + c;
                const bool in = s < N;
                const size_t sl = in ? s : N - 1;
#pragma unroll
                for (int kb = 0; kb < 4; ++kb) {
                    const float v = H1[sl * kH + 16 * kb + r];
                    h1[sb][kb][c] = in ? v : 0.f;
                }
                const float v2 = H2[sl * kH + unit];
                h2[sb][c] = in ? v2 : 0.f;
                const float e = Y[sl] - T[sl];
                dy[sb][c] = in ? scale * e : 0.f;
#pragma unroll
                for (int ib = 0; ib < 2; ++ib) {
                    const bool ok = in && 16 * ib + r < d;
                    const float v = X[sl * d + (16 * ib + r < d ? 16 * ib + r : 0)];
                    xt[sb][ib][c] = ok ? v : 0.f;
                }
            }
            const long long s = t0 + 16 * sb + r;
            const size_t sl = s < N ? s : N - 1;
#pragma unroll
            for (int jb = 0; jb < 4; ++jb) h2t[sb][jb] = row_piece(H2, sl, kH, 16 * jb + 4 * q);
            const float e = Y[sl] - T[sl];
            dyr[sb] = s < N ? scale * e : 0.f;
        }
#pragma unroll
        for (int sb = 0; sb < 2; ++sb) {
            f4m_t d2, d1 = zero;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                d2[c] = h2[sb][c] > 0.f ? dy[sb][c] * w3 : 0.f;
                gw3 = fmaf(dy[sb][c], h2[sb][c], gw3);
                gb3 += dy[sb][c];
                gb2 += d2[c];
            }
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) gW2[kb] = mlp_mma(d2, h1[sb][kb], gW2[kb]);
#pragma unroll
            for (int jb = 0; jb < 4; ++jb) {
                f4m_t m;
#pragma unroll
                for (int c = 0; c < 4; ++c) m[c] = h2t[sb][jb][c] > 0.f ? dyr[sb] * w3t[jb][c] : 0.f;
                d1 = mlp_mma(m, w2[jb], d1);
            }
            // the mask: this wavefront's own block of H1 (w is wave-uniform)
            const f4m_t own = w == 0 ? h1[sb][0] : w == 1 ? h1[sb][1] : w == 2 ? h1[sb][2] : h1[sb][3];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                d1[c] = own[c] > 0.f ? d1[c] : 0.f;
                gb1 += d1[c];
            }
            gW1[0] = mlp_mma(xt[sb][0], d1, gW1[0]);
            if (d > 16) gW1[1] = mlp_mma(xt[sb][1], d1, gW1[1]);
        }
    }
    float* out = part + (size_t)blockIdx.x * o.total;
#pragma unroll
    for (int ib = 0; ib < 2; ++ib)
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (16 * ib + 4 * q + c < d) out[o.W1 + unit * d + 16 * ib + 4 * q + c] = gW1[ib][c];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int c = 0; c < 4; ++c) out[o.W2 + (16 * w + 4 * q + c) * kH + 16 * kb + r] = gW2[kb][c];
    gb1 = sum_q(gb1);
    gb2 = sum_q(gb2);
    gw3 = sum_q(gw3);
    gb3 = sum_q(gb3);
    if (q == 0) {
        out[o.b1 + unit] = gb1;
        out[o.b2 + unit] = gb2;
        out[o.w3 + unit] = gw3;
        if (w == 0 && r == 0) out[o.b3] = gb3;
    }
}

// grad = sum of the partial vectors, each workgroup 64 parameters: sixteen
// wavefronts sum a segment of the blocks each (256-byte row pieces, at most 16
// loads a lane, all in flight) and the segments are added in order.  One
// thread per parameter walking every block took 31.0 us at 131 partials of
// 5249 parameters (21 workgroups, one chain of loads each), against 4.4 us now.
__global__ void __launch_bounds__(kRedParams* kRedSegs) mlp_reduce_k(int nblocks, int P, const float* __restrict__ part,
                                                                     float* __restrict__ grad) {
    __shared__ float seg[kRedSegs][kRedParams];
    const int w = wave_index(), lane = threadIdx.x & 63;
    const int i = blockIdx.x * kRedParams + lane;
    const int per = (nblocks + kRedSegs - 1) / kRedSegs;
    const float* p = part + (i < P ? i : 0);
    float s = 0.f;
    const int b1 = min(w * per + per, nblocks);
#pragma unroll 16
    for (int b = w * per; b < b1; ++b) s += p[(size_t)b * P];
    seg[w][lane] = s;
    __syncthreads();
    if (w == 0 && i < P) {
        float t = 0.f;
#pragma unroll
        for (int u = 0; u < kRedSegs; ++u) t += seg[u][lane];
        grad[i] = t;
    }
}

__global__ void __launch_bounds__(256) mlp_adam_k(int P, float* __restrict__ p, const float* __restrict__ g,
                                                  float* __restrict__ m, float* __restrict__ v, float lr, float b1,
                                                  float b2, float eps, float bc1, float bc2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= P) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
}

}  // namespace

size_t mlp_num_params(int d) { return (size_t)offsets(d).total; }

// Backward workgroups, one partial vector each: the launch and the workspace
// size both come from here.
static int mlp_backward_blocks(int N) {
    const long long tiles = ((long long)N + kBwdSamples - 1) / kBwdSamples;
    return (int)(tiles < kBwdBlocks ? tiles : kBwdBlocks);
}

size_t mlp_backward_workspace_bytes(int N, int d) {
    return sizeof(float) * (size_t)mlp_backward_blocks(N) * offsets(d).total;
}

int launch_mlp_forward(int N, int d, const float* X, const float* P, float* H1, float* H2, float* Y, void* stream) {
    (void)hipGetLastError();  // a stale error of an earlier runtime call is not ours
    const int nb = (int)(((long long)N + kFwdSamples - 1) / kFwdSamples);
    hipLaunchKernelGGL(mlp_forward_k, dim3(nb), dim3(256), 0, (hipStream_t)stream, N, d, X, P, H1, H2, Y);
    return (int)hipGetLastError();
}

int launch_mlp_backward(int N, int d, const float* X, const float* P, const float* H1, const float* H2,
                        const float* Y, const float* T, float* grad, void* workspace, void* stream) {
    (void)hipGetLastError();  // a stale error of an earlier runtime call is not ours
    const int nb = mlp_backward_blocks(N);
    const int np = offsets(d).total;
    float* part = reinterpret_cast<float*>(workspace);
    hipLaunchKernelGGL(mlp_backward_k, dim3(nb), dim3(256), 0, (hipStream_t)stream, N, d, X, P, H1, H2, Y, T, part);
    hipLaunchKernelGGL(mlp_reduce_k, dim3((np + kRedParams - 1) / kRedParams), dim3(kRedParams * kRedSegs), 0,
                       (hipStream_t)stream, nb, np, part, grad);
    return (int)hipGetLastError();
}

int launch_mlp_adam(int P, float* p, const float* g, float* m, float* v, float lr, float b1, float b2, float eps,
                    float bc1, float bc2, void* stream) {
    (void)hipGetLastError();  // a stale error of an earlier runtime call is not ours
    hipLaunchKernelGGL(mlp_adam_k, dim3((P + 255) / 256), dim3(256), 0, (hipStream_t)stream, P, p, g, m, v, lr, b1,
                       b2, eps, bc1, bc2);
    return (int)hipGetLastError();
}

}  // namespace glass
