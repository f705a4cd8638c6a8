// llr_mlp.hip -- warm-start network a(u, 1/L) for the Robbins-Monro iteration
// (the paper's initial values a_i-bar, Sec. 2.4, learned from converged a_k):
//   uh = (u - 0.6)/0.1, lh = (1/L - 0.0875)/0.0375
//   h1 = tanh(W1 x + b1)        64, FP32 vector units
//   h2 = tanh(W2 h1 + b2)       64x64: bfloat16 MFMA (FP32 accumulate) or FP32
//   a  = 1 + 0.1 (W3 h2 + b3)   FP32
// Parameter vector (4417 FP32): W1[64][2], b1, W2[64][64], b2, W3[64], b3.
// Training: mean squared error on a, full-batch Adam; gradients in FP32.
#include <hip/hip_runtime.h>

#include "llr_internal.hpp"

namespace llr {

constexpr int H = kMlpH;
constexpr int OW1 = 0, OB1 = OW1 + 2 * H, OW2 = OB1 + H, OB2 = OW2 + H * H, OW3 = OB2 + H, OB3 = OW3 + H;
constexpr int kRows = kMlpRows;   // samples per block
constexpr int kMB = 512;          // threads per block
constexpr int HP = H + 4;         // row stride in LDS: 16 rows of 16-byte reads touch every bank once

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ short to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);   // round to nearest even
    return (short)(u >> 16);
}

// The network and one block of samples in LDS.
struct Net {
    float w1[2 * H], b1[H], b2[H], w3[H], b3;
    alignas(16) float w2[H][HP];
    __device__ float& at(int e) {
        if (e < OB1) return w1[e - OW1];
        if (e < OW2) return b1[e - OB1];
        if (e < OB2) return w2[(e - OW2) / H][(e - OW2) % H];
        if (e < OW3) return b2[e - OB2];
        if (e < OB3) return w3[e - OW3];
        return b3;
    }
};
struct Chunk {
    alignas(16) float h1[kRows][HP];
    alignas(16) float h2[kRows][HP];
    float x[kRows][2];
    float y[kRows];
};

// Forward of rows [0, nr) of a block of samples.
__device__ void fwd_chunk(const Net& w, Chunk& c, const float* __restrict__ u, const float* __restrict__ invL, int row0,
                          int nr, int bf16) {
    const int t = threadIdx.x;
    if (t < kRows) {
        c.x[t][0] = t < nr ? (u[row0 + t] - 0.6f) / 0.1f : 0.f;
        c.x[t][1] = t < nr ? (invL[row0 + t] - 0.0875f) / 0.0375f : 0.f;
    }
    __syncthreads();
    for (int e = t; e < kRows * H; e += kMB) {
        const int i = e / H, j = e - i * H;
        float v = 0.f;
        if (i < nr) v = tanhf(w.w1[2 * j] * c.x[i][0] + w.w1[2 * j + 1] * c.x[i][1] + w.b1[j]);
        c.h1[i][j] = v;
    }
    __syncthreads();
    if (bf16) {
        // v_mfma_f32_16x16x16_bf16 tiles, A[i][k] = h1, B[k][j] = W2[j][k]: wave wv
        // computes rows 16 (wv / 2) .. + 15 of the 32 columns from 32 (wv % 2)
        const int lane = t & 63, wv = t >> 6;
        const int li = lane & 15, kq = lane >> 4;
        const int rt = 16 * (wv >> 1);
        bf16x4 av[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const f32x4 f = *reinterpret_cast<const f32x4*>(&c.h1[rt + li][16 * ks + 4 * kq]);
#pragma unroll
            for (int r = 0; r < 4; ++r) av[ks][r] = to_bf16(f[r]);
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int j = 32 * (wv & 1) + 16 * q + li;
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const f32x4 f = *reinterpret_cast<const f32x4*>(&w.w2[j][16 * ks + 4 * kq]);
                bf16x4 bv;
#pragma unroll
                for (int r = 0; r < 4; ++r) bv[r] = to_bf16(f[r]);
                acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(av[ks], bv, acc, 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) c.h2[rt + 4 * kq + r][j] = tanhf(acc[r] + w.b2[j]);
        }
    } else {
        // 2 rows x 4 columns per thread, the sum over k in order
        const int jg = t & 15, i0 = 2 * (t >> 4);
        float z[2][4];
#pragma unroll
        for (int q = 0; q < 4; ++q) z[0][q] = z[1][q] = w.b2[jg + 16 * q];
#pragma unroll 2
        for (int k = 0; k < H; k += 4) {
            const f32x4 a0 = *reinterpret_cast<const f32x4*>(&c.h1[i0][k]);
            const f32x4 a1 = *reinterpret_cast<const f32x4*>(&c.h1[i0 + 1][k]);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 b = *reinterpret_cast<const f32x4*>(&w.w2[jg + 16 * q][k]);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    z[0][q] += b[r] * a0[r];
                    z[1][q] += b[r] * a1[r];
                }
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            c.h2[i0][jg + 16 * q] = tanhf(z[0][q]);
            c.h2[i0 + 1][jg + 16 * q] = tanhf(z[1][q]);
        }
    }
    __syncthreads();
    if (t < kRows) {
        float y = w.b3;
#pragma unroll 4
        for (int k = 0; k < H; k += 4) {
            const f32x4 h = *reinterpret_cast<const f32x4*>(&c.h2[t][k]);
#pragma unroll
            for (int r = 0; r < 4; ++r) y += w.w3[k + r] * h[r];
        }
        c.y[t] = y;
    }
    __syncthreads();
}

__global__ __launch_bounds__(kMB) void k_mlp_forward(const float* __restrict__ w, const float* __restrict__ u,
                                                      const float* __restrict__ invL, int n, int bf16,
                                                      double* __restrict__ a_out) {
    __shared__ Net net;
    __shared__ Chunk c;
    for (int e = threadIdx.x; e < kMlpNP; e += kMB) net.at(e) = w[e];
    const int row0 = blockIdx.x * kRows;
    const int nr = min(kRows, n - row0);
    fwd_chunk(net, c, u, invL, row0, nr, bf16);
    if ((int)threadIdx.x < nr) a_out[row0 + threadIdx.x] = 1.0 + 0.1 * (double)c.y[threadIdx.x];
}

// The samples' gradient sums of the chunks, in chunk order.
__device__ __forceinline__ float grad_sum(const float* __restrict__ part, int nchunk, int i) {
    float g = 0.f;
    for (int b = 0; b < nchunk; ++b) g += part[(size_t)b * kMlpNP + i];
    return g;
}
// Adam (Kingma & Ba), step t >= 1, of one parameter
__device__ __forceinline__ float adam_step(float w, float m, float v, float g, float c1, float c2, float lr, float& mo,
                                           float& vo) {
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    // explicit fused multiply-adds: both kernels round alike
    const float mi = __fmaf_rn(b1, m, (1.f - b1) * g);
    const float vi = __fmaf_rn(b2, v, (1.f - b2) * g * g);
    mo = mi;
    vo = vi;
    w -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    return w;
}

// Loss and gradient of one block of kRows samples (one block of threads per
// chunk), written as that chunk's partial sums; the sums over a chunk's samples
// and then over the chunks run in a fixed order.  With t >= 1 the kernel first
// takes Adam step t from the previous launch's partial sums: every block
// updates its own copy of the parameters in LDS, block 0 writes them (and the
// moments) to the other buffer, so an epoch is one launch.
//
// One chunk's gradient is 4 x 64^3 multiply-adds.  A single block of 256 threads
// that walked all chunks with one LDS read per operand took 182 us an epoch at
// 160 samples (LDS-issue bound), and the Adam launch 4.7 us.  Here the chunks
// run in parallel and a thread computes 2 x 4 outputs of each matrix product
// from 16-byte LDS reads, 8 multiply-adds per 3 reads of 4 values or fewer:
// 187 -> 16.7 us an epoch at 160 samples, 4300 -> 31.6 at 4096 (bfloat16).
// What is left is one block's latency: the Adam step's loads, two tanh layers
// and the two 64^3 products of one CU.
__global__ __launch_bounds__(kMB) void k_mlp_epoch(MlpBuf in, MlpBuf out, const float* __restrict__ part_in, int t_adam,
                                                    float lr, const float* __restrict__ u,
                                                    const float* __restrict__ invL, const double* __restrict__ a, int n,
                                                    int bf16, float* __restrict__ part_out,
                                                    double* __restrict__ loss_out) {
    __shared__ Net net;
    __shared__ Chunk c;
    __shared__ alignas(16) float d2[kRows][HP];
    __shared__ float dy[kRows];
    __shared__ double lpart[kRows];
    const int t = threadIdx.x, nchunk = (int)gridDim.x, b = (int)blockIdx.x;
    constexpr int PT = (kMlpNP + kMB - 1) / kMB;   // parameters per thread
    if (t_adam > 0) {
        const float c1 = 1.f - powf(0.9f, (float)t_adam), c2 = 1.f - powf(0.999f, (float)t_adam);
        float gs[PT], w0[PT], m0[PT], v0[PT];
        // every load of a chunk's row is in flight at once: the rows were written
        // on other XCDs a moment ago, so each round trip is a long one
#pragma unroll
        for (int q = 0; q < PT; ++q) {
            const int e = min(t + q * kMB, kMlpNP - 1);
            gs[q] = 0.f;
            w0[q] = in.w[e];
            m0[q] = in.m[e];
            v0[q] = in.v[e];
        }
#pragma unroll 4
        for (int k = 0; k < nchunk; ++k)
#pragma unroll
            for (int q = 0; q < PT; ++q) gs[q] += part_in[(size_t)k * kMlpNP + min(t + q * kMB, kMlpNP - 1)];
#pragma unroll
        for (int q = 0; q < PT; ++q) {
            const int e = t + q * kMB;
            if (e >= kMlpNP) break;
            float mo, vo;
            const float wn = adam_step(w0[q], m0[q], v0[q], gs[q], c1, c2, lr, mo, vo);
            net.at(e) = wn;
            if (b == 0) {
                out.w[e] = wn;
                out.m[e] = mo;
                out.v[e] = vo;
            }
        }
    } else {
#pragma unroll
        for (int q = 0; q < PT; ++q) {
            const int e = t + q * kMB;
            if (e < kMlpNP) net.at(e) = in.w[e];
        }
    }
    const int row0 = b * kRows;
    const int nr = min(kRows, n - row0);
    float* __restrict__ g = part_out + (size_t)b * kMlpNP;
    fwd_chunk(net, c, u, invL, row0, nr, bf16);
    if (t < kRows) {
        float r = 0.f;
        double rr = 0.0;
        if (t < nr) {
            rr = (1.0 + 0.1 * (double)c.y[t]) - a[row0 + t];
            r = (float)rr;
        }
        lpart[t] = rr * rr;
        dy[t] = 2.f * r / (float)n * 0.1f;
    }
    __syncthreads();
    for (int e = t; e < kRows * H; e += kMB) {
        const int i = e / H, k = e - i * H;
        d2[i][k] = i < nr ? dy[i] * net.w3[k] * (1.f - c.h2[i][k] * c.h2[i][k]) : 0.f;
    }
    // (tanh(0 w + b2) in the rows past the last sample: not a number for an infinite w)
    if (nr < kRows)
        for (int e = nr * H + t; e < kRows * H; e += kMB) c.h2[e / H][e % H] = 0.f;
    __syncthreads();
    // output layer, biases and the loss, on a wavefront each; the rows past the
    // last sample hold zeros (dy, h2, d2, d1, lpart), so every sum runs over all rows
    // with its loads issued ahead
    if (t < H) {
        float s = 0.f;
#pragma unroll 16
        for (int i = 0; i < kRows; ++i) s += dy[i] * c.h2[i][t];
        g[OW3 + t] = s;
    } else if (t < 2 * H) {
        float s = 0.f;
#pragma unroll 16
        for (int i = 0; i < kRows; ++i) s += d2[i][t - H];
        g[OB2 + t - H] = s;
    } else if (t == 2 * H) {
        float s = 0.f;
#pragma unroll 16
        for (int i = 0; i < kRows; ++i) s += dy[i];
        g[OB3] = s;
    } else if (t == 3 * H) {
        double s = 0.0;
#pragma unroll 16
        for (int i = 0; i < kRows; ++i) s += lpart[i];
        loss_out[b] = s / (double)n;
    }
    // hidden layer 2: dW2[j][k] = sum_i d2[i][j] h1[i][k]
    {
        const int k0 = 4 * (t & 15), j0 = 2 * (t >> 4);
        float s[2][4] = {};
#pragma unroll 4
        for (int i = 0; i < kRows; ++i) {
            const f32x4 h = *reinterpret_cast<const f32x4*>(&c.h1[i][k0]);
            const f32x2 d = *reinterpret_cast<const f32x2*>(&d2[i][j0]);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[0][r] += d[0] * h[r];
                s[1][r] += d[1] * h[r];
            }
        }
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) g[OW2 + H * (j0 + q) + k0 + r] = s[q][r];
    }
    // back to layer 1: d1[i][k] = (sum_j W2[j][k] d2[i][j]) (1 - h1^2); reuse c.h2 as d1
    float s1[2][4] = {};
    const int k0 = 4 * (t & 15), i0 = 2 * (t >> 4);
#pragma unroll 2
    for (int j = 0; j < H; j += 4) {
        const f32x4 da = *reinterpret_cast<const f32x4*>(&d2[i0][j]);
        const f32x4 db = *reinterpret_cast<const f32x4*>(&d2[i0 + 1][j]);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f32x4 w = *reinterpret_cast<const f32x4*>(&net.w2[j + q][k0]);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s1[0][r] += w[r] * da[q];
                s1[1][r] += w[r] * db[q];
            }
        }
    }
    __syncthreads();   // the output layer's sums over c.h2 are done
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int i = i0 + q;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            c.h2[i][k0 + r] = i < nr ? s1[q][r] * (1.f - c.h1[i][k0 + r] * c.h1[i][k0 + r]) : 0.f;
    }
    __syncthreads();
    if (t < H) {
        float s = 0.f;
#pragma unroll 16
        for (int i = 0; i < kRows; ++i) s += c.h2[i][t];
        g[OB1 + t] = s;
    } else if (t < 2 * H) {
        float s = 0.f;
#pragma unroll 16
        for (int i = 0; i < kRows; ++i) s += c.h2[i][t - H] * c.x[i][0];
        g[OW1 + 2 * (t - H)] = s;
    } else if (t < 3 * H) {
        float s = 0.f;
#pragma unroll 16
        for (int i = 0; i < kRows; ++i) s += c.h2[i][t - 2 * H] * c.x[i][1];
        g[OW1 + 2 * (t - 2 * H) + 1] = s;
    }
}

// Adam step t of all parameters from the chunks' partial sums, or (t = 0) the
// gradient itself into out.w
__global__ void k_mlp_adam(MlpBuf in, MlpBuf out, const float* __restrict__ part, int nchunk, int t, float lr) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kMlpNP) return;
    const float g = grad_sum(part, nchunk, i);
    if (t == 0) {
        out.w[i] = g;
        return;
    }
    const float c1 = 1.f - powf(0.9f, (float)t), c2 = 1.f - powf(0.999f, (float)t);
    float mo, vo;
    out.w[i] = adam_step(in.w[i], in.m[i], in.v[i], g, c1, c2, lr, mo, vo);
    out.m[i] = mo;
    out.v[i] = vo;
}

// loss of each epoch from its chunks' parts, in chunk order
__global__ void k_mlp_loss(const double* __restrict__ part, int nchunk, int epochs, double* __restrict__ loss) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= epochs) return;
    double s = 0.0;
    for (int b = 0; b < nchunk; ++b) s += part[(size_t)e * nchunk + b];
    loss[e] = s;
}

// Xavier-uniform weights from Philox (kind 4, w0 = parameter index), zero biases.
__global__ void k_mlp_init(uint32_t k0, uint32_t k1, float* __restrict__ w) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kMlpNP) return;
    double lim = 0.0;
    if (i < OB1) lim = sqrt(6.0 / (2 + H));
    else if (i >= OW2 && i < OB2) lim = sqrt(6.0 / (H + H));
    else if (i >= OW3 && i < OB3) lim = sqrt(6.0 / (H + 1));
    if (lim == 0.0) { w[i] = 0.f; return; }
    const uint4 r = philox10(make_uint4((uint32_t)i, ctr1_word(0, 0, kMlp, 0), 0u, 0u), k0, k1);
    const double uu = ((double)r.x + 0.5) * 0x1p-32;
    w[i] = (float)__fma_rn(2.0 * lim, uu, -lim);
}

void launch_mlp_init(uint64_t seed, float* w, hipStream_t st) {
    hipLaunchKernelGGL(k_mlp_init, dim3((kMlpNP + 255) / 256), dim3(256), 0, st, (uint32_t)seed,
                       (uint32_t)(seed >> 32), w);
}
void launch_mlp_forward(const float* w, const float* u, const float* invL, int n, int bf16, double* a_out,
                        hipStream_t st) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_mlp_forward, dim3((n + kRows - 1) / kRows), dim3(kMB), 0, st, w, u, invL, n, bf16, a_out);
}
void launch_mlp_epoch(MlpBuf in, MlpBuf out, const float* part_in, int t_adam, float lr, const float* u,
                      const float* invL, const double* a, int n, int bf16, float* part_out, double* loss_part,
                      hipStream_t st) {
    hipLaunchKernelGGL(k_mlp_epoch, dim3((unsigned)mlp_chunks(n)), dim3(kMB), 0, st, in, out, part_in, t_adam, lr, u,
                       invL, a, n, bf16, part_out, loss_part);
}
void launch_mlp_adam(MlpBuf in, MlpBuf out, const float* part, int n, int t, float lr, hipStream_t st) {
    hipLaunchKernelGGL(k_mlp_adam, dim3((kMlpNP + 255) / 256), dim3(256), 0, st, in, out, part, mlp_chunks(n), t, lr);
}
void launch_mlp_loss(const double* loss_part, int n, int epochs, double* loss, hipStream_t st) {
    hipLaunchKernelGGL(k_mlp_loss, dim3((unsigned)((epochs + 255) / 256)), dim3(256), 0, st, loss_part, mlp_chunks(n),
                       epochs, loss);
}

}  // namespace llr
