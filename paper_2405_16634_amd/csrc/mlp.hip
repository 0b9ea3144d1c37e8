// The neighbourhood MLP of the learned warm start: 48 -> 64 -> 64 -> 3 with
// ReLU, BF16 operands and FP32 accumulation, inference and training.
//
// One kernel (k_mlp) runs the whole network on tiles of 32 rows, one
// wavefront per tile, on the CDNA4 matrix cores (v_mfma_f32_16x16x32_bf16),
// and for training also the loss, the backward pass and the tile's part of
// the parameter gradients, which stay in accumulators until the wavefront's
// last tile.  Lane l (r = l % 16, q = l / 16) holds A[r][8q+i] and B[8q+i][r],
// i = 0..7, and receives C[4q+i][r], i = 0..3.  The layers are computed
// transposed, outputs x rows (A = W^T, kept in registers; B = the rows'
// activations), so that a lane's four outputs of one row are consecutive: they
// go to LDS row by row, where the next layer's B fragments are 16-byte reads,
// and, for the gradients (sums over the 32 rows: one MFMA per 16x16 tile),
// column by column.
//
// What bounds it: nothing but the rows themselves has to be read (192 + 12
// bytes each, 13 MB at 64k rows), so it is the latency of a wavefront's chain
// of loads, LDS exchanges and 92 MFMAs per tile.  One GEMM launch per product,
// each reading FP32 activations through strides and writing them back, with
// one workgroup per bias gradient, took 16 launches and 590 us for a training
// step on 64k rows, and 116 us for 100k rows of inference (1184 us for 1M);
// this takes 32 us, and 17 us (63 us for 1M, 3.2 TB/s).
//
// Operands are rounded to BF16 (round to nearest even) when fragments are
// formed; sums are FP32.  The parameter gradients are added over the tiles of
// a wavefront, its workgroup's wavefronts and the workgroups in a fixed order,
// so training is reproducible bit for bit.
//
// Parameter vector (FP32 master copy, 7491 values): W1 [48][64], b1 [64],
// W2 [64][64], b2 [64], W3 [64][3], b3 [3]; row-major [in][out].
#include <float.h>
#include <string.h>

#include <algorithm>

#include "common.h"
#include "internal.h"

namespace wnnc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// FP32 -> BF16, round to nearest even (the hardware conversion).
__device__ inline __bf16 to_bf16(float f) { return (__bf16)f; }

constexpr int kMlpWaves = 4;    // wavefronts per workgroup
constexpr int kMlpTile = 32;    // rows per wavefront and step
constexpr int kMlpMaxWgs = 256; // training: workgroups (one partial gradient each)
// LDS strides (BF16 values) of a row's 64 outputs and of a column's 32 rows;
// multiples of 16 bytes that spread the lanes over the banks.
constexpr int kRowStride = 72, kColStride = 40;

struct MlpArgs {
    const float *P;       // parameters
    const float *X;       // n x 48
    const float *L;       // labels (training), n x 3
    float *Y;             // outputs (inference), n x 3
    float *part;          // training: kMlpParams per workgroup
    double *lpart;        // training: loss sum of each workgroup
    int64_t n;
    float inv_n;
    int aligned;          // X is 16-byte aligned
};

// Eight FP32 values as a BF16 fragment.
__device__ inline bf16x8 frag8(const float *v) {
    bf16x8 f;
#pragma unroll
    for (int i = 0; i < 8; ++i) f[i] = to_bf16(v[i]);
    return f;
}

__device__ inline bf16x8 ld_frag(const __bf16 *p) { return *(const bf16x8 *)p; }

// Keeps the compiler from moving a wavefront's own LDS accesses (which execute
// in order) across this point.
__device__ inline void lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ inline f32x4 mma(const bf16x8 &a, const bf16x8 &b, const f32x4 &c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

template <bool TRAIN>
__global__ __launch_bounds__(kMlpWaves *kWave, TRAIN ? 1 : 2) void k_mlp(MlpArgs g) {
    __shared__ float sp[kMlpParams];
    // per wavefront: the activations row by row and, for training, the
    // features, hidden activations, their gradients and the outputs' column by
    // column; at the end the wavefront's gradient
    constexpr int kLds = kMlpTile * kRowStride +
                         (TRAIN ? (kMlpIn + 4 * kMlpHidden + 16) * kColStride : 0);
    static_assert(!TRAIN || kLds * sizeof(__bf16) >= kMlpParams * sizeof(float), "gradient fits");
    __shared__ __attribute__((aligned(16))) __bf16 work[kMlpWaves][kLds];
    __shared__ double lsum[kMlpWaves];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int r = lane & 15, q = lane >> 4;
    {  // all of a thread's loads in flight at once
        constexpr int kPer = (kMlpParams + kMlpWaves * kWave - 1) / (kMlpWaves * kWave);
        float v[kPer];
#pragma unroll
        for (int i = 0; i < kPer; ++i)
            v[i] = g.P[min(tid + i * kMlpWaves * kWave, kMlpParams - 1)];
#pragma unroll
        for (int i = 0; i < kPer; ++i)
            if (tid + i * kMlpWaves * kWave < kMlpParams) sp[tid + i * kMlpWaves * kWave] = v[i];
    }
    __syncthreads();

    // weight fragments: forward A[out][in], backward A[in][out]
    bf16x8 w1[4][2], w2[4][2], w3[2], v3[4], v2[4][2];
    float b1[4][4], b2[4][4], b3[3];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            float a1[8], a2[8], c2[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int in = 32 * k + 8 * q + i, out = 16 * m + r;
                a1[i] = in < kMlpIn ? sp[kOffW1 + in * kMlpHidden + out] : 0.f;
                a2[i] = sp[kOffW2 + in * kMlpHidden + out];
                c2[i] = TRAIN ? sp[kOffW2 + out * kMlpHidden + in] : 0.f;
            }
            w1[m][k] = frag8(a1);
            w2[m][k] = frag8(a2);
            if (TRAIN) v2[m][k] = frag8(c2);
        }
        float c3[8];
#pragma unroll
        for (int i = 0; i < 8; ++i)
            c3[i] = TRAIN && q == 0 && i < kMlpOut ? sp[kOffW3 + (16 * m + r) * kMlpOut + i] : 0.f;
        if (TRAIN) v3[m] = frag8(c3);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            b1[m][i] = sp[kOffB1 + 16 * m + 4 * q + i];
            b2[m][i] = sp[kOffB2 + 16 * m + 4 * q + i];
        }
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        float a3[8];
#pragma unroll
        for (int i = 0; i < 8; ++i)
            a3[i] = r < kMlpOut ? sp[kOffW3 + (32 * k + 8 * q + i) * kMlpOut + r] : 0.f;
        w3[k] = frag8(a3);
    }
#pragma unroll
    for (int i = 0; i < kMlpOut; ++i) b3[i] = sp[kOffB3 + i];

    constexpr int kCols = kMlpHidden * kColStride;
    __bf16 *rm = work[wv], *h1t = rm + kMlpTile * kRowStride, *h2t = h1t + kCols,
           *d1t = h2t + kCols, *d2t = d1t + kCols, *xt = d2t + kCols,
           *yt = xt + kMlpIn * kColStride;  // (all but rm in training only)
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 gw1[3][4], gw2[4][4], gw3[4];
    float gb1[4][4], gb2[4][4], gb3[3] = {0.f, 0.f, 0.f};
    double loss = 0.0;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        gw3[m] = zero;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (m < 3) gw1[m][k] = zero;
            gw2[m][k] = zero;
            gb1[m][k] = gb2[m][k] = 0.f;
        }
    }
    if (TRAIN) {  // the outputs beyond the third stay zero
        for (int i = lane; i < 16 * kColStride; i += kWave) yt[i] = to_bf16(0.f);
    }

    // a 64 x 32 layer output (outputs x rows): to LDS row by row
    auto put_rows = [&](const f32x4 (&h)[4][2]) {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                bf16x4 o;
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] = to_bf16(h[m][t][i]);
                *(bf16x4 *)(rm + (16 * t + r) * kRowStride + 16 * m + 4 * q) = o;
            }
        }
    };
    // and column by column
    auto put_cols = [&](__bf16 *c, const f32x4 (&h)[4][2]) {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    c[(16 * m + 4 * q + i) * kColStride + 16 * t + r] = to_bf16(h[m][t][i]);
            }
        }
    };

    const int64_t tiles = (g.n + kMlpTile - 1) / kMlpTile;
    for (int64_t tile = (int64_t)blockIdx.x * kMlpWaves + wv; tile < tiles;
         tile += (int64_t)gridDim.x * kMlpWaves) {
        const int64_t row0 = tile * kMlpTile;
        // layer 1: the rows' features, 8 consecutive ones per lane
        f32x4 h1[4][2], h2[4][2];
#pragma unroll
        for (int m = 0; m < 4; ++m) h1[m][0] = h1[m][1] = h2[m][0] = h2[m][1] = zero;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int64_t row = row0 + 16 * t + r;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int f0 = 32 * k + 8 * q;
                float v[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = 0.f;
                if (row < g.n && f0 < kMlpIn) {
                    const float *xp = g.X + row * kMlpIn + f0;
                    if (g.aligned) {
                        const float4 u0 = *(const float4 *)xp, u1 = *(const float4 *)(xp + 4);
                        v[0] = u0.x, v[1] = u0.y, v[2] = u0.z, v[3] = u0.w;
                        v[4] = u1.x, v[5] = u1.y, v[6] = u1.z, v[7] = u1.w;
                    } else {
#pragma unroll
                        for (int i = 0; i < 8; ++i) v[i] = xp[i];
                    }
                }
                const bf16x8 b = frag8(v);
#pragma unroll
                for (int m = 0; m < 4; ++m) h1[m][t] = mma(w1[m][k], b, h1[m][t]);
                if (TRAIN && f0 < kMlpIn) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) xt[(f0 + i) * kColStride + 16 * t + r] = b[i];
                }
            }
        }
#pragma unroll
        for (int m = 0; m < 4; ++m) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
#pragma unroll
                for (int i = 0; i < 4; ++i) h1[m][t][i] = fmaxf(h1[m][t][i] + b1[m][i], 0.f);
            }
        }
        put_rows(h1);
        if (TRAIN) put_cols(h1t, h1);
        lds_order();
        // layer 2
#pragma unroll
        for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const bf16x8 b = ld_frag(rm + (16 * t + r) * kRowStride + 32 * k + 8 * q);
#pragma unroll
                for (int m = 0; m < 4; ++m) h2[m][t] = mma(w2[m][k], b, h2[m][t]);
            }
        }
#pragma unroll
        for (int m = 0; m < 4; ++m) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
#pragma unroll
                for (int i = 0; i < 4; ++i) h2[m][t][i] = fmaxf(h2[m][t][i] + b2[m][i], 0.f);
            }
        }
        lds_order();
        put_rows(h2);
        if (TRAIN) put_cols(h2t, h2);
        lds_order();
        // layer 3: lanes of q = 0 hold the three outputs of their row
        bf16x8 dy[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            f32x4 y = zero;
#pragma unroll
            for (int k = 0; k < 2; ++k)
                y = mma(w3[k], ld_frag(rm + (16 * t + r) * kRowStride + 32 * k + 8 * q), y);
            const int64_t row = row0 + 16 * t + r;
            const float y0 = y[0] + b3[0], y1 = y[1] + b3[1], y2 = y[2] + b3[2];
            const bool in = q == 0 && row < g.n;
            if (!TRAIN) {
                if (in) g.Y[3 * row] = y0, g.Y[3 * row + 1] = y1, g.Y[3 * row + 2] = y2;
                continue;
            }
            // loss = mean_i (1 - cos(y_i, l_i)) and its gradient
            float d[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            if (in) {
                const float l0 = g.L[3 * row], l1 = g.L[3 * row + 1], l2 = g.L[3 * row + 2];
                const float yy = sqrtf(y0 * y0 + y1 * y1 + y2 * y2);
                const float ll = sqrtf(l0 * l0 + l1 * l1 + l2 * l2);
                float cs = 0.f;
                if (yy > 0.f && ll > 0.f) {
                    const float yl = y0 * l0 + y1 * l1 + y2 * l2;
                    cs = yl / (yy * ll);
                    // d cos / d y = l/(|y||l|) - (y.l) y / (|y|^3 |l|)
                    const float a = 1.0f / (yy * ll), b = yl / (yy * yy * yy * ll);
                    d[0] = -g.inv_n * (l0 * a - y0 * b);
                    d[1] = -g.inv_n * (l1 * a - y1 * b);
                    d[2] = -g.inv_n * (l2 * a - y2 * b);
                }
                loss += 1.0 - (double)cs;
            }
            dy[t] = frag8(d);
            if (q == 0) {
#pragma unroll
                for (int o = 0; o < kMlpOut; ++o) {
                    gb3[o] += d[o];
                    yt[o * kColStride + 16 * t + r] = dy[t][o];
                }
            }
        }
        if constexpr (TRAIN) {
            // back through layer 3 and the ReLUs
            f32x4 d2[4][2], d1[4][2];
#pragma unroll
            for (int m = 0; m < 4; ++m) {
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    d2[m][t] = mma(v3[m], dy[t], zero);
                    d1[m][t] = zero;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if (!(h2[m][t][i] > 0.f)) d2[m][t][i] = 0.f;
                        gb2[m][i] += d2[m][t][i];
                    }
                }
            }
            lds_order();
            put_rows(d2);
            put_cols(d2t, d2);
            lds_order();
#pragma unroll
            for (int t = 0; t < 2; ++t) {
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const bf16x8 b = ld_frag(rm + (16 * t + r) * kRowStride + 32 * k + 8 * q);
#pragma unroll
                    for (int m = 0; m < 4; ++m) d1[m][t] = mma(v2[m][k], b, d1[m][t]);
                }
            }
#pragma unroll
            for (int m = 0; m < 4; ++m) {
#pragma unroll
                for (int t = 0; t < 2; ++t) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if (!(h1[m][t][i] > 0.f)) d1[m][t][i] = 0.f;
                        gb1[m][i] += d1[m][t][i];
                    }
                }
            }
            put_cols(d1t, d1);
            lds_order();
            // the weight gradients: sums over the tile's 32 rows
            bf16x8 fa[4], fb[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                if (m < 3) fa[m] = ld_frag(xt + (16 * m + r) * kColStride + 8 * q);
                fb[m] = ld_frag(d1t + (16 * m + r) * kColStride + 8 * q);
            }
#pragma unroll
            for (int m = 0; m < 3; ++m) {
#pragma unroll
                for (int k = 0; k < 4; ++k) gw1[m][k] = mma(fa[m], fb[k], gw1[m][k]);
            }
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                fa[m] = ld_frag(h1t + (16 * m + r) * kColStride + 8 * q);
                fb[m] = ld_frag(d2t + (16 * m + r) * kColStride + 8 * q);
            }
#pragma unroll
            for (int m = 0; m < 4; ++m) {
#pragma unroll
                for (int k = 0; k < 4; ++k) gw2[m][k] = mma(fa[m], fb[k], gw2[m][k]);
            }
            const bf16x8 fy = ld_frag(yt + r * kColStride + 8 * q);
#pragma unroll
            for (int m = 0; m < 4; ++m)
                gw3[m] = mma(ld_frag(h2t + (16 * m + r) * kColStride + 8 * q), fy, gw3[m]);
        }
        lds_order();
    }
    if constexpr (TRAIN) {
        // bias sums over the 16 rows of a lane group; the loss over the lanes
#pragma unroll
        for (int d = 8; d > 0; d >>= 1) {
#pragma unroll
            for (int m = 0; m < 4; ++m) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    gb1[m][i] += __shfl_xor(gb1[m][i], d, kWave);
                    gb2[m][i] += __shfl_xor(gb2[m][i], d, kWave);
                }
            }
#pragma unroll
            for (int o = 0; o < kMlpOut; ++o) gb3[o] += __shfl_xor(gb3[o], d, kWave);
            loss += __shfl_xor(loss, d, kWave);
        }
        if (lane == 0) lsum[wv] = loss;
        // the workgroup's gradient: its wavefronts' in order
        float *mine = (float *)work[wv];
        lds_order();
#pragma unroll
        for (int m = 0; m < 4; ++m) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int in = 16 * m + 4 * q + i;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (m < 3) mine[kOffW1 + in * kMlpHidden + 16 * k + r] = gw1[m][k][i];
                    mine[kOffW2 + in * kMlpHidden + 16 * k + r] = gw2[m][k][i];
                }
                if (r < kMlpOut) mine[kOffW3 + in * kMlpOut + r] = gw3[m][i];
                if (r == 0) {
                    mine[kOffB1 + in] = gb1[m][i];
                    mine[kOffB2 + in] = gb2[m][i];
                }
            }
        }
        if (lane == 0) {
#pragma unroll
            for (int o = 0; o < kMlpOut; ++o) mine[kOffB3 + o] = gb3[o];
        }
        __syncthreads();
        float *out = g.part + (int64_t)blockIdx.x * kMlpParams;
        for (int i = tid; i < kMlpParams; i += kMlpWaves * kWave) {
            float v = ((const float *)work[0])[i];
#pragma unroll
            for (int w = 1; w < kMlpWaves; ++w) v += ((const float *)work[w])[i];
            out[i] = v;
        }
        if (tid == 0) {
            double s = 0.0;
            for (int w = 0; w < kMlpWaves; ++w) s += lsum[w];
            g.lpart[blockIdx.x] = s;
        }
    }
}

// grad[p] = the sum of the workgroups' partial gradients, in a fixed order:
// four wavefronts of a workgroup take every fourth partial of 64 parameters.
__global__ __launch_bounds__(256) void k_param_sum(const float *__restrict__ part, int count,
                                                   float *__restrict__ grad) {
    __shared__ float sh[4][kWave];
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    const int p = blockIdx.x * kWave + lane;
    float s = 0.f;
    if (p < kMlpParams) {
        constexpr int kUnroll = 16;
        for (int w0 = wv; w0 < count; w0 += 4 * kUnroll) {
            float v[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                // (beyond the last partial: the last one, not added)
                const int w = w0 + 4 * u;
                v[u] = part[(int64_t)(w < count ? w : count - 1) * kMlpParams + p];
            }
#pragma unroll
            for (int u = 0; u < kUnroll; ++u)
                if (w0 + 4 * u < count) s += v[u];
        }
    }
    sh[wv][lane] = s;
    __syncthreads();
    if (wv == 0 && p < kMlpParams) grad[p] = ((s + sh[1][lane]) + sh[2][lane]) + sh[3][lane];
}

__global__ __launch_bounds__(256) void k_unit_rows(const float *__restrict__ Y, int64_t n,
                                                   float *__restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float y0 = Y[3 * i], y1 = Y[3 * i + 1], y2 = Y[3 * i + 2];
    const float yy = sqrtf(y0 * y0 + y1 * y1 + y2 * y2);
    const float f = yy > 0.f ? 1.0f / yy : 0.0f;
    out[3 * i] = y0 * f, out[3 * i + 1] = y1 * f, out[3 * i + 2] = y2 * f;
}

// Adam on the FP32 master parameters (bias-corrected moments).
__global__ __launch_bounds__(256) void k_adam(float *__restrict__ p, float *__restrict__ m,
                                              float *__restrict__ v,
                                              const float *__restrict__ g, int count, float lr,
                                              float b1, float b2, float eps, float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// ------------------------------------------------------------------ host --

static MlpArgs mlp_args(const float *P, const float *X, int64_t n) {
    MlpArgs g;
    memset(&g, 0, sizeof(g));
    g.P = P;
    g.X = X;
    g.n = n;
    g.aligned = ((uintptr_t)X & 15) == 0 ? 1 : 0;
    return g;
}

static int64_t mlp_wgs(int64_t n) {
    const int64_t per = (int64_t)kMlpTile * kMlpWaves;
    return (n + per - 1) / per;
}

hipError_t mlp_forward(wnnc_ctx_s *ctx, const float *P, const float *X, int64_t n, float *Y) {
    MlpArgs g = mlp_args(P, X, n);
    g.Y = Y;
    // (three workgroups per CU fit the LDS)
    const int64_t wgs = std::min<int64_t>(mlp_wgs(n), 3 * kMlpMaxWgs);
    hipLaunchKernelGGL((k_mlp<false>), dim3((unsigned)wgs), dim3(kMlpWaves * kWave), 0, ctx->stream,
                       g);
    return hipGetLastError();
}

hipError_t mlp_normals(wnnc_ctx_s *ctx, const float *Y, int64_t n, float *out) {
    hipLaunchKernelGGL(k_unit_rows, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, ctx->stream, Y,
                       n, out);
    return hipGetLastError();
}

hipError_t mlp_loss_grad(wnnc_ctx_s *ctx, const float *P, const float *X, const float *L,
                         int64_t n, float *grad, double *loss) {
    hipStream_t st = ctx->stream;
    const int64_t wgs = std::min<int64_t>(mlp_wgs(n), kMlpMaxWgs);
    hipError_t e = ctx->mlp_part.ensure(wgs * kMlpParams);
    if (e == hipSuccess) e = ctx->mlp_lpart.ensure(wgs);
    if (e != hipSuccess) return e;
    MlpArgs g = mlp_args(P, X, n);
    g.L = L;
    g.part = ctx->mlp_part.p;
    g.lpart = ctx->mlp_lpart.p;
    g.inv_n = 1.0f / (float)n;
    hipLaunchKernelGGL((k_mlp<true>), dim3((unsigned)wgs), dim3(kMlpWaves * kWave), 0, st, g);
    hipLaunchKernelGGL(k_param_sum, dim3((kMlpParams + kWave - 1) / kWave), dim3(256), 0, st,
                       ctx->mlp_part.p, (int)wgs, grad);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (loss) {
        std::vector<double> lp((size_t)wgs);
        e = hipMemcpyAsync(lp.data(), ctx->mlp_lpart.p, (size_t)wgs * sizeof(double),
                           hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) return e;
        double s = 0.0;
        for (double v : lp) s += v;
        *loss = s / (double)n;
    }
    return hipSuccess;
}

hipError_t mlp_adam(wnnc_ctx_s *ctx, float *P, float *m, float *v, const float *g, int step,
                    float lr, float b1, float b2, float eps) {
    const float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3((kMlpParams + 255) / 256), dim3(256), 0, ctx->stream, P, m, v,
                       g, kMlpParams, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

}  // namespace wnnc
