// Learned radial force filter f(|k|, a) = 1 + g(|k|/k_Nyq, a), g a 2-64-64-1
// perceptron with SiLU activations (pmwd paper, Statement of Need: learned
// components running with the simulation, spatial optimisation of the PM
// gravity solver), evaluated on every integer |n|^2 of the mesh once per force
// evaluation, its backward pass, and Adam.
//
// Parameter vector (4417 FP32): W1[64][2] | b1[64] | W2[64][64] | b2[64] |
// W3[1][64] | b3[1], output index first.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.h"

namespace pmx {
namespace {

constexpr int HID = 64;
constexpr int OW1 = 0, OB1 = 128, OW2 = 192, OB2 = 4288, OW3 = 4352, OB3 = 4416, NPAR = 4417;

__device__ __forceinline__ float sigmoid(float z) { return 1.f / (1.f + expf(-z)); }

// Sum over the 64 lanes of a wave (every lane gets the total).
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// features of integer |n|^2: |k| / k_Nyq = 2 sqrt(n2) / n
__device__ __forceinline__ float feature0(long n2, int n) {
    return 2.f * sqrtf((float)n2) / (float)n;
}

// A work-group of four waves per 64 |n|^2 entries, one lane per entry in each:
// wave w computes first-layer units 16w .. 16w+15 (passed to the others through
// LDS) and then second-layer units 16w .. 16w+15; wave 0 adds the output layer.
// The weights are the same for all lanes and come through scalar loads, so the
// inner product is one vector instruction per weight with nothing read from LDS.
// Bound by the vector ALUs (4160 FMAs and 128 SiLUs per entry; an FMA costs a
// SiLU's thirtieth).  One lane per entry with the weights read from LDS took
// 47 us for the 12289 entries of a 128^3 mesh (192 waves on 1024 SIMDs) and
// 100 us for the 196609 of 512^3 (LDS reads); this takes 16.5 and 54 us, and 34 us
// for the tables of nine scale factors at 128^3 (blockIdx.y: the table).  Every
// sum runs over its inputs in index order.
__global__ void __launch_bounds__(256)
k_mlp_table(const float* __restrict__ theta, int n, ScaleFactors sf, float fscale, long ntab,
            long stride, float* __restrict__ radial, float* __restrict__ table) {
    __shared__ float hs[HID][64];   // first-layer units, then second-layer terms, by entry
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const float a = sf.a[blockIdx.y];
    for (long e0 = (long)blockIdx.x * 64; e0 < ntab; e0 += (long)gridDim.x * 64) {
        const long e = e0 + lane;
        const float x0 = feature0(e < ntab ? e : 0, n), x1 = a;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int i = 16 * w + k;
            const float z1 = theta[OW1 + 2 * i] * x0 + theta[OW1 + 2 * i + 1] * x1 + theta[OB1 + i];
            hs[i][lane] = z1 * sigmoid(z1);
        }
        __syncthreads();
        float h1[HID];
#pragma unroll
        for (int i = 0; i < HID; ++i) h1[i] = hs[i][lane];
        __syncthreads();
#pragma unroll 4
        for (int k = 0; k < 16; ++k) {
            const int o = 16 * w + k;
            const float* wr = theta + OW2 + o * HID;
            float z = theta[OB2 + o];
#pragma unroll
            for (int i = 0; i < HID; ++i) z += wr[i] * h1[i];
            hs[o][lane] = z * sigmoid(z);
        }
        __syncthreads();
        if (w == 0) {
            float g = theta[OB3];
#pragma unroll
            for (int o = 0; o < HID; ++o) g += theta[OW3 + o] * hs[o][lane];
            const float f = 1.f + g;
            if (e < ntab) {
                const long o = blockIdx.y * stride + e;
                if (table) table[o] = f;
                if (radial) radial[o] = e == 0 ? 0.f : f * fscale / (float)e;
            }
        }
        __syncthreads();   // hs is rewritten by the next entries
    }
}

constexpr int kChunk = 64;   // table entries per tile
constexpr int kBwdBlocks = 256;

typedef float v16f __attribute__((ext_vector_type(16)));

// D += A B on the FP32 matrix cores, A 32 x 64, B 64 x 32, D 32 x 32, with
// a(k) and b(k) this lane's A[lane % 32][k] and B[k][lane % 32] for k = 2 step +
// lane / 32.  Element r of D sits in row mfma_row(r, lane), column lane % 32.
template <class FA, class FB>
__device__ __forceinline__ v16f mfma64(v16f d, FA a, FB b) {
#pragma unroll
    for (int s = 0; s < 32; ++s) d = __builtin_amdgcn_mfma_f32_32x32x2f32(a(s), b(s), d, 0, 0, 0);
    return d;
}
__device__ __forceinline__ int mfma_row(int r, int lane) {
    return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
}

// Block-partial dL/dtheta for dL/df = fbar over the table; partials to scratch.
// Per chunk of 64 entries the second layer is three 64 x 64 x 64 products, on
// the FP32 matrix cores, each of the four waves taking a 32 x 32 quadrant:
//   Z2 = W2 H1,   dW2 += dZ2 H1^T,   dH1 = W2^T dZ2
// (H1, dZ2 and dH1 are [unit][entry], in LDS rows of 65 so that rows and columns
// are both free of bank conflicts; W2 stays in registers in both layouts).  The
// first layer is one lane per entry, wave w holding units 16w .. 16w+15.  On the
// vector units the products read up to two LDS words per FMA: 352 us for the
// 196609 entries of a 512^3 mesh and 36 us for the 12289 of 128^3; now 110 and
// 21 us.  Sums over entries stay in registers until the last chunk, in a fixed
// order.
__global__ void __launch_bounds__(256)
k_mlp_bwd(const float* __restrict__ theta, int n, ScaleFactors sf, long ntab, long stride,
          int nchunks, const float* __restrict__ fbar, float* __restrict__ scratch) {
    constexpr int PL = kChunk + 1;
    static_assert(kChunk == 64 && HID == 64, "one entry per lane, four 32 x 32 quadrants");
    __shared__ float h1s[HID * PL];    // H1, then dH1
    __shared__ float dz2s[HID * PL];
    __shared__ float red[2][2][HID];   // db2 and dW3 by column half
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int mh = 32 * (w >> 1), nh = 32 * (w & 1);   // the wave's quadrant
    const int c = lane & 31, kh = lane >> 5;
    float w2[32], w2t[32];   // W2[mh + c][.] and W2[.][mh + c] at k = 2 s + kh
#pragma unroll
    for (int s = 0; s < 32; ++s) {
        w2[s] = theta[OW2 + (mh + c) * HID + 2 * s + kh];
        w2t[s] = theta[OW2 + (2 * s + kh) * HID + mh + c];
    }
    v16f dw2 = {0.f};
    float db2[16], dw3[16], dw1[16][3], db3 = 0.f;
#pragma unroll
    for (int k = 0; k < 16; ++k) db2[k] = dw3[k] = dw1[k][0] = dw1[k][1] = dw1[k][2] = 0.f;
    for (int q = blockIdx.x; q < nchunks * sf.n; q += gridDim.x) {
        const int t = q / nchunks;   // the table of this chunk
        const long c0 = (long)(q - t * nchunks) * kChunk;
        const float a = sf.a[t];
        // first layer at entry c0 + lane
        const long e = c0 + lane;
        const float x0 = feature0(e < ntab ? e : 0, n), x1 = a;
        float ds1[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int i = 16 * w + k;
            const float z = theta[OW1 + 2 * i] * x0 + theta[OW1 + 2 * i + 1] * x1 + theta[OB1 + i];
            const float sg = sigmoid(z);
            h1s[i * PL + lane] = z * sg;
            ds1[k] = sg * (1.f + z * (1.f - sg));
        }
        // dL/df at this lane's column of the second layer's quadrant
        const long ec = c0 + nh + c;
        const float dg = ec < ntab ? fbar[t * stride + ec] : 0.f;
        if (mh == 0 && kh == 0) db3 += dg;
        __syncthreads();
        v16f z2 = {0.f};
        z2 = mfma64(z2, [&](int s) { return w2[s]; },
                    [&](int s) { return h1s[(2 * s + kh) * PL + nh + c]; });
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int o = mh + mfma_row(r, lane);
            const float z = z2[r] + theta[OB2 + o];
            const float sg = sigmoid(z);
            const float dz = dg * theta[OW3 + o] * (sg * (1.f + z * (1.f - sg)));
            dw3[r] += dg * (z * sg);
            db2[r] += dz;
            dz2s[o * PL + nh + c] = dz;
        }
        __syncthreads();
        dw2 = mfma64(dw2, [&](int s) { return dz2s[(mh + c) * PL + 2 * s + kh]; },
                     [&](int s) { return h1s[(nh + c) * PL + 2 * s + kh]; });
        v16f dh = {0.f};
        dh = mfma64(dh, [&](int s) { return w2t[s]; },
                    [&](int s) { return dz2s[(2 * s + kh) * PL + nh + c]; });
        __syncthreads();   // H1 has been read
#pragma unroll
        for (int r = 0; r < 16; ++r) h1s[(mh + mfma_row(r, lane)) * PL + nh + c] = dh[r];
        __syncthreads();
        // a thread's own slots: the next chunk's first layer may overwrite them
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const float dz = h1s[(16 * w + k) * PL + lane] * ds1[k];
            dw1[k][0] += dz * x0;
            dw1[k][1] += dz * x1;
            dw1[k][2] += dz;
        }
    }
    float* out = scratch + (long)blockIdx.x * NPAR;
#pragma unroll
    for (int r = 0; r < 16; ++r)
        out[OW2 + (mh + mfma_row(r, lane)) * HID + nh + c] = dw2[r];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int i = 16 * w + k;
        const float s0 = wave_sum(dw1[k][0]), s1 = wave_sum(dw1[k][1]), s2 = wave_sum(dw1[k][2]);
        if (lane == 0) {
            out[OW1 + 2 * i] = s0;
            out[OW1 + 2 * i + 1] = s1;
            out[OB1 + i] = s2;
        }
    }
    // second-layer biases and output weights: over the 32 columns, then the halves
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        float sb = db2[r], sw = dw3[r];
#pragma unroll
        for (int o = 1; o < 32; o <<= 1) {
            sb += __shfl_xor(sb, o);
            sw += __shfl_xor(sw, o);
        }
        if (c == 0) {
            red[w & 1][0][mh + mfma_row(r, lane)] = sb;
            red[w & 1][1][mh + mfma_row(r, lane)] = sw;
        }
    }
    db3 = wave_sum(db3);
    __syncthreads();
    if (threadIdx.x < HID) {
        out[OB2 + threadIdx.x] = red[0][0][threadIdx.x] + red[1][0][threadIdx.x];
        out[OW3 + threadIdx.x] = red[0][1][threadIdx.x] + red[1][1][threadIdx.x];
    }
    __syncthreads();
    if (w < 2 && lane == 0) red[w][0][0] = db3;   // waves 0 and 1 hold the two halves
    __syncthreads();
    if (threadIdx.x == 0) out[OB3] = red[0][0][0] + red[1][0][0];
}

// gtheta += the block partials, 64 parameters per work-group: each of the 16
// waves adds every 16th block's partials (eight loads in flight), then the
// waves' sums are added in order.  (One thread per parameter added all the
// blocks one load after the other: 47 us for 193 blocks, 62 us for 256; now
// under 5 us.)
__global__ void __launch_bounds__(1024)
k_mlp_reduce(const float* __restrict__ scratch, int nblocks, float* __restrict__ gtheta) {
    __shared__ float part[16][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int p = blockIdx.x * 64 + lane;
    const int pc = p < NPAR ? p : NPAR - 1;
    float s = 0.f;
    int b = w;
    for (; b + 7 * 16 < nblocks; b += 8 * 16) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = scratch[(long)(b + 16 * u) * NPAR + pc];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; b < nblocks; b += 16) s += scratch[(long)b * NPAR + pc];
    part[w][lane] = s;
    __syncthreads();
    if (w == 0 && p < NPAR) {
        float t = 0.f;
#pragma unroll
        for (int k = 0; k < 16; ++k) t += part[k][lane];
        gtheta[p] += t;
    }
}

__global__ void __launch_bounds__(256)
k_adam(float* __restrict__ p, const float* __restrict__ g, int ngrad, float* __restrict__ m,
       float* __restrict__ v, int n, float lr, float b1, float b2, float eps, float bc1,
       float bc2) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    float gi = 0.f;  // mean of the batch of gradients, summed in a fixed order
    for (int j = 0; j < ngrad; ++j) gi += g[(long)j * n + i];
    gi /= (float)ngrad;
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
}

}  // namespace

long mlp_backward_scratch(int) { return (long)kBwdBlocks * NPAR; }

void launch_mlp_table(const float* theta, int n, const ScaleFactors& sf, float fscale, long stride,
                      float* radial, float* table, hipStream_t s) {
    const long ntab = 3L * (n / 2) * (n / 2) + 1;
    long nb = (ntab + 63) / 64;
    if (nb > 4096) nb = 4096;
    hipLaunchKernelGGL(k_mlp_table, dim3((unsigned)nb, sf.n), dim3(256), 0, s, theta, n, sf, fscale,
                       ntab, stride, radial, table);
}

void launch_mlp_backward(const float* theta, int n, const ScaleFactors& sf, long stride,
                         const float* fbar, float* gtheta, float* scratch, hipStream_t s) {
    const long ntab = 3L * (n / 2) * (n / 2) + 1;
    const int nchunks = (int)((ntab + kChunk - 1) / kChunk);
    const int nb = std::min(nchunks * sf.n, kBwdBlocks);
    hipLaunchKernelGGL(k_mlp_bwd, dim3(nb), dim3(256), 0, s, theta, n, sf, ntab, stride, nchunks,
                       fbar, scratch);
    hipLaunchKernelGGL(k_mlp_reduce, dim3((NPAR + 63) / 64), dim3(1024), 0, s, scratch, nb, gtheta);
}

void launch_adam(float* p, const float* g, int ngrad, float* m, float* v, int n, float lr,
                 float b1, float b2, float eps, float bc1, float bc2, hipStream_t s) {
    hipLaunchKernelGGL(k_adam, dim3((n + 255) / 256), dim3(256), 0, s, p, g, ngrad, m, v, n, lr,
                       b1, b2, eps, bc1, bc2);
}

}  // namespace pmx
