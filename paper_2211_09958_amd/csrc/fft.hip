// Batched 3-D real FFT passes for gfx950 and the fused Fourier-space Poisson
// gradient (and its transpose).
//
// A 3-D transform is three passes over HBM, one per axis:
//   * last axis (contiguous rows): a real row of n samples is read as n/2
//     complex pairs, transformed with an n/2-point complex FFT, and split into
//     the n/2 + 1 half-spectrum values with the standard post-twiddle
//         X[k] = (Z[k] + Z*[n/2-k]) / 2 - i W^k (Z[k] - Z*[n/2-k]) / 2;
//   * axes 1 and 0 (strided): a work-group loads an n x W tile (W consecutive
//     columns, each row segment W*8 bytes) and transforms the W columns
//     together, exchanging through LDS between Stockham stages.  Rows are
//     stored in the blocked order of layout.h, which keeps both strided passes
//     within a few dozen pages.
// The Poisson multiply F~_j = i k_j f(|k|) delta_k / k^2 is fused into the
// axis-0 pass: one load of the spectrum, one forward column FFT, then for each
// j a multiply and inverse column FFT straight to the output buffer, so the
// spectrum is read once and each gradient component written once.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "fft_engine.h"
#include "kernels.h"
#include "layout.h"
#include "xcd.h"

namespace pmx {
namespace {

// Non-temporal store of one complex value (the last-axis passes write data that
// no later pass reads before the whole buffer has streamed through the caches;
// measured 3 % faster there, 7 % slower in the strided passes).
__device__ __forceinline__ void st_nt(float2* p, float2 v) {
    __builtin_nontemporal_store(v.x, &p->x);
    __builtin_nontemporal_store(v.y, &p->y);
}
__device__ __forceinline__ float2 ld_nt(const float2* p) {
    return make_float2(__builtin_nontemporal_load(&p->x), __builtin_nontemporal_load(&p->y));
}
// The same for a pair of floats of any 4-byte alignment (a caller's array).
__device__ __forceinline__ float2 ld_nt_pair(const float* p) {
    return make_float2(__builtin_nontemporal_load(p), __builtin_nontemporal_load(p + 1));
}
__device__ __forceinline__ void st_nt_pair(float* p, float2 v) {
    __builtin_nontemporal_store(v.x, p);
    __builtin_nontemporal_store(v.y, p + 1);
}

// Plain row number i0 n + i1 of storage row r (layout.h).
__device__ __forceinline__ long plain_row(long r, int n) {
    int i0, i1;
    mesh_row_inv(r, n, i0, i1);
    return (long)i0 * n + i1;
}

// Lanes-per-transform and values-per-lane choices per transform length.
template <int H>
struct Cfg {
    static constexpr int E = fft_values_per_lane(H);
    static constexpr int T = H / E;
    // columns per work-group for strided passes (8 columns = 64-byte row
    // segments; XCD-aware numbering keeps both halves of a 128-byte line on
    // the same L2)
    static constexpr int W = H >= 512 ? 8 : 16;
    // columns of the plain strided passes: at 512 points two work-groups of 16
    // columns (full 128-byte lines, 1024 threads) fit on a CU, 252 -> 227 us per
    // 512^3 pass; the passes with a second transform or stream keep 8 (split
    // 380 -> 434 us, merge 376 -> 402 with 16)
    static constexpr int WS = H == 512 ? 16 : W;
    // minimum waves per SIMD requested from the compiler (caps VGPRs so that
    // two work-groups fit on a CU for the large transforms)
    static constexpr int MINW = H >= 512 ? 4 : 1;
    static constexpr int ROWS = T >= 256 ? 1 : 256 / T;   // rows per work-group, last axis
    // columns per work-group for the axis-1 split pass: with two output
    // streams, half-written 128-byte lines leave L2 before the neighbouring tile
    // writes their other half (writes 1.24x the bytes at 8 columns), so the
    // 1024-point split takes 16 columns, full lines (one 1024-thread
    // work-group per CU, as the LDS holds one)
    static constexpr int WY = H >= 1024 ? 16 : W;
};

// ---------------------------------------------------------- last axis

// DENSE: the real rows are read from a caller's [N][N][N] array in plain row
// order (any 4-byte alignment) instead of from the buffer itself, so a
// caller's mesh needs no copy into the workspace layout first.  That copy moved
// as many bytes as the pass and took longer (512^3: 411 us for the copy, 218 us
// for the pass).  With all four layout copies folded into the first and last
// passes, a 512^3 R2C plus C2R takes 1.76 ms instead of 2.75 ms.
template <int N, bool DENSE>
__global__ void __launch_bounds__(Cfg<N / 2>::T * Cfg<N / 2>::ROWS)
k_fft_x_r2c(const float* __restrict__ real, float2* __restrict__ buf, int cs, long nrows,
            long bufStride, const float2* __restrict__ tw, int ntw,
            const float2* __restrict__ st) {
    constexpr int H = N / 2, E = Cfg<H>::E, T = Cfg<H>::T, ROWS = Cfg<H>::ROWS;
    constexpr int LS = lds_slots(H);
    __shared__ float2 lds[ROWS * LS];
    const int r = threadIdx.x / T, j = threadIdx.x % T;
    const long row = (long)xcd_block(blockIdx.x, gridDim.x) * ROWS + r;
    const bool valid = row < nrows;
    float2* rowp = buf + blockIdx.y * bufStride + (valid ? row : 0) * cs;
    const int twN = ntw / N;
    // rowp points at row 0 for rows past the end, so every load is in bounds
    // and none sits in a branch (which would make each wait for its data)
    float2 v[E];
    const float* src = reinterpret_cast<const float*>(rowp);
    if constexpr (DENSE) src = real + plain_row(valid ? row : 0, N) * N;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        v[e] = ld_nt_pair(src + 2 * (j + e * T));
        if (!valid) v[e] = make_float2(0.f, 0.f);
    }
    float2* L = lds + r * LS;
    fft_lds<H, E, -1>(v, L, 1, 0, j, st);
    __syncthreads();
    if (!valid) return;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int k = j + e * T;
        float2 zk = L[lpad(k)], zc = cconj(L[lpad((H - k) & (H - 1))]);
        float2 A = cadd(zk, zc), B = csub(zk, zc);
        float2 w = tw[k * twN];
        float2 iwB = cmul_i<1>(cmul(w, B));
        float2 X = make_float2(0.5f * (A.x - iwB.x), 0.5f * (A.y - iwB.y));
        if (k == 0) {
            X = make_float2(zk.x + zk.y, 0.f);
            st_nt(&rowp[H], make_float2(zk.x - zk.y, 0.f));
        }
        st_nt(&rowp[k], X);
    }
}

// kmul_buf >= 0: the spectrum of buffer kmul_buf is first multiplied by i k2
// (zero on the Nyquist column), i.e. this pass also takes the spectral
// derivative along the last axis.  DENSE: the real rows go to a caller's
// [N][N][N] array in plain row order (as in k_fft_x_r2c).  OPEN: unless *open is 0
// (an instance of its own: a test of the pointer cost the smallest meshes 0.2 us).
template <int N, bool DENSE, bool OPEN>
__global__ void __launch_bounds__(Cfg<N / 2>::T * Cfg<N / 2>::ROWS)
k_fft_x_c2r(float2* __restrict__ buf, float* __restrict__ real, const int* __restrict__ open, int cs,
            long nrows, long bufStride, int kmul_buf, const float2* __restrict__ tw, int ntw,
            const float2* __restrict__ st) {
    constexpr int H = N / 2, E = Cfg<H>::E, T = Cfg<H>::T, ROWS = Cfg<H>::ROWS;
    constexpr int LS = lds_slots(H);
    __shared__ float2 lds[ROWS * LS];
    const int r = threadIdx.x / T, j = threadIdx.x % T;
    const long row = (long)xcd_block(blockIdx.x, gridDim.x) * ROWS + r;
    const bool valid = row < nrows;
    float2* rowp = buf + blockIdx.y * bufStride + (valid ? row : 0) * cs;
    const int twN = ntw / N;
    float2* L = lds + r * LS;
    const bool kmul = (int)blockIdx.y == kmul_buf;
    const bool store = !OPEN || *open != 0;
    // rowp points at row 0 for rows past the end, so every load is in bounds
    // and none sits in a branch (which would make each wait for its data)
    float2 x[E];
#pragma unroll
    for (int e = 0; e < E; ++e) x[e] = ld_nt(&rowp[j + e * T]);
    const float2 xh = ld_nt(&rowp[H]);
    // the pre-twiddles, loaded with the row (a load after the barrier below
    // would be waited for there)
    float2 twk[E];
#pragma unroll
    for (int e = 0; e < E; ++e) twk[e] = tw[(j + e * T) * twN];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int k = j + e * T;
        float2 y = valid ? x[e] : make_float2(0.f, 0.f);
        if (kmul) y = make_float2(-(float)k * y.y, (float)k * y.x);
        L[lpad(k)] = y;
    }
    if (j == 0) L[lpad(H)] = (valid && !kmul) ? xh : make_float2(0.f, 0.f);
    __syncthreads();
    float2 v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int k = j + e * T;
        float2 xk = L[lpad(k)], xc = cconj(L[lpad(H - k)]);
        float2 A = cadd(xk, xc), B = cmulc(csub(xk, xc), twk[e]);
        v[e] = cadd(A, cmul_i<1>(B));
    }
    __syncthreads();
    fft_lds<H, E, 1>(v, L, 1, 0, j, st);
    __syncthreads();
    if (!valid || !store) return;
    float* dst = reinterpret_cast<float*>(rowp);
    if constexpr (DENSE) dst = real + plain_row(row, N) * N;
#pragma unroll
    for (int e = 0; e < E; ++e) st_nt_pair(dst + 2 * (j + e * T), L[lpad(j + e * T)]);
}

__device__ __forceinline__ int signed_freq(int p, int n) { return p < n / 2 ? p : p - n; }

// ---------------------------------------------------------- strided axes

// Tile t -> (a, cb): columns cb*W .. cb*W+W-1 of the rows with the other slow
// index fixed to a; element p of the transform sits in mesh row (a, p) for
// AXIS = 1 and (p, a) for AXIS = 0 (storage order: layout.h).
// `spec`, with SPEC: a caller's dense half spectrum [H][H][H/2+1] (AXIS = 0),
// which the forward pass writes and the inverse pass reads in place of the
// buffer, so that no separate pass changes the layout (512^3: 251 us each way).
template <int H, int DIR, int AXIS, bool SPEC>
__global__ void __launch_bounds__(Cfg<H>::T * Cfg<H>::WS, Cfg<H>::MINW)
k_fft_strided(float2* __restrict__ buf, typename std::conditional<DIR < 0, float2*, const float2*>::type
              __restrict__ spec, int cs, int ncb, long bufStride, const float2* __restrict__ st) {
    static_assert(!SPEC || AXIS == 0, "dense spectra are the first or last pass, along axis 0");
    constexpr int E = Cfg<H>::E, T = Cfg<H>::T, W = Cfg<H>::WS;
    __shared__ float2 lds[lds_slots(H) * W];
    const int c = threadIdx.x % W, j = threadIdx.x / W;
    const int tile = (int)xcd_block(blockIdx.x, gridDim.x);
    const int a = tile / ncb, cb = tile % ncb;
    float2* base = buf + blockIdx.y * bufStride + cb * W + c;
    auto at = [&](int p) -> float2& {
        return base[(AXIS == 1 ? mesh_row(a, p, H) : mesh_row(p, a, H)) * cs];
    };
    // dense element p of the column: row (p, a), column k2 (one past the half
    // spectrum is padding, loaded from column H/2 and replaced by zero)
    const int k2 = cb * W + c;
    const bool stored = k2 <= H / 2;
    auto dense = [&](int p) -> long {
        return ((long)p * H + a) * (H / 2 + 1) + (stored ? k2 : H / 2);
    };
    float2 v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        if constexpr (SPEC && DIR > 0) {
            v[e] = spec[dense(j + e * T)];
            if (!stored) v[e] = make_float2(0.f, 0.f);
        } else {
            v[e] = at(j + e * T);
        }
    }
    fft_lds<H, E, DIR>(v, lds, W, c, j, st);
    __syncthreads();
    if constexpr (SPEC && DIR < 0) {
        if (!stored) return;
#pragma unroll
        for (int e = 0; e < E; ++e) spec[dense(j + e * T)] = lds[lpad(j + e * T) * W + c];
    } else {
#pragma unroll
        for (int e = 0; e < E; ++e) at(j + e * T) = lds[lpad(j + e * T) * W + c];
    }
}

// Inverse axis-1 pass that splits G into the two spectra it feeds: out_g =
// IFFT_1(G) (F~_2 = i k2 times it, applied by the last-axis C2R) and, in place,
// F~_1 = IFFT_1(i n1 G) (zero on the Nyquist plane of axis 1).  The column is
// loaded once and held in registers for the second transform (a reload misses
// L2: the other work-groups stream several times its size through it in
// between); the stage twiddles come from an LDS copy, which leaves the
// registers for it.
template <int H>
__global__ void __launch_bounds__(Cfg<H>::T * Cfg<H>::WY, Cfg<H>::MINW)
k_fft_y_split(float2* __restrict__ g, float2* __restrict__ out_g, int cs, int ncb,
              const float2* __restrict__ st) {
    constexpr int E = Cfg<H>::E, T = Cfg<H>::T, W = Cfg<H>::WY;
    // exchange buffer | the H-point part of the stage-twiddle table (H - 1 entries)
    __shared__ float2 lds[lds_slots(H) * W + H];
    float2* tab = lds + lds_slots(H) * W;
    // read first in the second stage, after the first stage's barrier
    for (int i = threadIdx.x; i < H - 1; i += T * W) tab[i] = st[H + i];
    const int c = threadIdx.x % W, j = threadIdx.x / W;
    const int tile = (int)xcd_block(blockIdx.x, gridDim.x);
    const int a = tile / ncb, cb = tile % ncb;   // a: axis-0 index
    const int k2 = cb * W + c;
    auto off = [&](int p) -> long { return mesh_row(a, p, H) * cs + k2; };
    float2 x[E], v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        x[e] = g[off(j + e * T)];
        v[e] = x[e];
    }
    fft_lds_tab<H, E, 1>(v, lds, W, c, j, tab);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) out_g[off(j + e * T)] = lds[lpad(j + e * T) * W + c];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int p = j + e * T;
        const float f1 = p == H / 2 ? 0.f : (float)signed_freq(p, H);
        v[e] = make_float2(-f1 * x[e].y, f1 * x[e].x);
    }
    __syncthreads();   // every lane has read the first transform's output
    fft_lds_tab<H, E, 1>(v, lds, W, c, j, tab);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) g[off(j + e * T)] = lds[lpad(j + e * T) * W + c];
}

// Forward axis-1 pass of the transposed gradient that merges the axis-1 and
// axis-2 terms: g1 <- n1 FFT_1(g1) + n2 FFT_1(g2), with n1 the axis-1 frequency
// of the output row (zero on its Nyquist plane) and n2 = k2 the column's
// (zero on its Nyquist column).  Both factors are known once the axis-1
// transform is done and stay fixed along axis 0, so the axis-0 pass reads this
// one spectrum in place of two.  The g1 column's transform is held in
// registers while g2's is taken; the g2 column is loaded with g1's, and the
// stage twiddles come from an LDS copy (as in k_fft_y_split).
template <int H>
__global__ void __launch_bounds__(Cfg<H>::T * Cfg<H>::WY, Cfg<H>::MINW)
k_fft_y_merge(float2* __restrict__ g1, const float2* __restrict__ g2, int cs, int ncb,
              const float2* __restrict__ st) {
    constexpr int E = Cfg<H>::E, T = Cfg<H>::T, W = Cfg<H>::WY;
    __shared__ float2 lds[lds_slots(H) * W + H];
    float2* tab = lds + lds_slots(H) * W;
    // read first in the second stage, after the first stage's barrier
    for (int i = threadIdx.x; i < H - 1; i += T * W) tab[i] = st[H + i];
    const int c = threadIdx.x % W, j = threadIdx.x / W;
    const int tile = (int)xcd_block(blockIdx.x, gridDim.x);
    const int a = tile / ncb, cb = tile % ncb;   // a: axis-0 index
    const int k2 = cb * W + c;
    const float f2 = k2 == H / 2 ? 0.f : (float)k2;
    auto off = [&](int p) -> long { return mesh_row(a, p, H) * cs + k2; };
    float2 x[E], v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        v[e] = g1[off(j + e * T)];
        x[e] = g2[off(j + e * T)];
    }
    fft_lds_tab<H, E, -1>(v, lds, W, c, j, tab);
    __syncthreads();
    float2 h[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int p = j + e * T;
        const float f1 = p == H / 2 ? 0.f : (float)signed_freq(p, H);
        const float2 y = lds[lpad(p) * W + c];
        h[e] = make_float2(f1 * y.x, f1 * y.y);
        v[e] = x[e];
    }
    __syncthreads();   // every lane has read the first transform's output
    fft_lds_tab<H, E, -1>(v, lds, W, c, j, tab);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int p = j + e * T;
        const float2 y = lds[lpad(p) * W + c];
        g1[off(p)] = make_float2(h[e].x + f2 * y.x, h[e].y + f2 * y.y);
    }
}

// Axis-0 pass with a 2LPT multiplier (launch_fft_z_mul).  A multiplier pass of
// its own read and wrote the spectrum once more: 50 us per use at 256^3, for 24 us
// of transform.
struct LptMul {
    int a, b, mode, accumulate;
    const float* table;
    float scale;
};

// The factor of mode (i0, i1, k2).
template <int H>
__device__ __forceinline__ float lpt_factor(const LptMul& M, int i0, int i1, int k2) {
    const int nv[3] = {signed_freq(i0, H), signed_freq(i1, H), k2};
    const bool nyq[3] = {i0 == H / 2, i1 == H / 2, k2 == H / 2};
    const int m2 = nv[0] * nv[0] + nv[1] * nv[1] + nv[2] * nv[2];
    if (m2 == 0 || k2 > H / 2) return 0.f;
    const int na = M.a == 0 ? nv[0] : (M.a == 1 ? nv[1] : nv[2]);
    const int nb = M.b == 0 ? nv[0] : (M.b == 1 ? nv[1] : nv[2]);
    const bool za = M.a == 0 ? nyq[0] : (M.a == 1 ? nyq[1] : nyq[2]);
    const bool zb = M.b == 0 ? nyq[0] : (M.b == 1 ? nyq[1] : nyq[2]);
    const float r = M.table ? M.table[m2] : 1.f / (float)m2;
    float w;
    if (M.mode == 0) w = M.a != M.b && (za || zb) ? 0.f : (float)(na * nb) * r;
    else if (M.mode == 1) w = (float)(m2 - na * na) * r;
    else w = (float)m2 * r;
    return w * M.scale;
}

template <int H, int DIR>
__global__ void __launch_bounds__(Cfg<H>::T * Cfg<H>::W, Cfg<H>::MINW)
k_fft_z_mul(const float2* __restrict__ src, float2* __restrict__ dst, int cs, int ncb, LptMul M,
            const float2* __restrict__ st) {
    constexpr int E = Cfg<H>::E, T = Cfg<H>::T, W = Cfg<H>::W;
    __shared__ float2 lds[lds_slots(H) * W];
    const int c = threadIdx.x % W, j = threadIdx.x / W;
    const int tile = (int)xcd_block(blockIdx.x, gridDim.x);
    const int i1 = tile / ncb, k2 = (tile % ncb) * W + c;
    auto off = [&](int p) -> long { return mesh_row(p, i1, H) * cs + k2; };
    float2 v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = src[off(j + e * T)];
    if constexpr (DIR > 0) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const float w = lpt_factor<H>(M, j + e * T, i1, k2);
            v[e] = make_float2(w * v[e].x, w * v[e].y);
        }
    }
    fft_lds<H, E, DIR>(v, lds, W, c, j, st);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int q = j + e * T;
        float2 y = lds[lpad(q) * W + c];
        if constexpr (DIR < 0) {
            const float w = lpt_factor<H>(M, q, i1, k2);
            y.x *= w;
            y.y *= w;
            if (M.accumulate) {
                const float2 d = dst[off(q)];
                y.x += d.x;
                y.y += d.y;
            }
        }
        dst[off(q)] = y;
    }
}

// ---------------------------------------------------------- planes

// Both transforms of a plane i0 = const (axes 2 and 1) by one work-group, the
// plane's half spectrum staying in LDS between them, for meshes up to
// kMaxPlane.  These are bound by launches and by the latency of each pass (a
// launch costs the host 3-4 us; a pass over the 2 MB of a 64^3 mesh runs 3.5-5
// us), so one launch in place of two or three is what counts: 7.2 us for the
// force meshes' inverse of 64^3 instead of 3.4 + 4.6 + 5.2, 9.8 us for the
// cotangents' merged forward instead of 4.6 + 3.6 + 4.5.  At 128^3 a plane takes
// 72 KB of LDS, there are 128 of them for 256 CUs, and the fused forms take
// 28-34 us where the separate passes take 26-27: no gain; at 256^3 a plane does
// not fit in LDS.
template <int N>
struct Plane {
    static constexpr int H = N / 2, PW = H + 1;          // complex row length, columns
    static constexpr int EX = fft_values_per_lane(H), TX = H / EX;
    static constexpr int EY = fft_values_per_lane(N), TY = N / EY;
    // every row, and every column, has its lanes
    static constexpr int NT = ((PW * TY > N * TX ? PW * TY : N * TX) + 63) / 64 * 64;
    static constexpr int LS = lds_slots(H);
    static constexpr int SLOTS = N * LS > lds_slots(N) * PW ? N * LS : lds_slots(N) * PW;
    // lanes without a row or column transform one of this region's, which nobody
    // reads (a branch around their stores changes which products the compiler
    // contracts, and with it the last bits of every transform)
    static constexpr int ALL = NT > N * TX || NT > PW * TY ? 2 * SLOTS : SLOTS;
    // M[lpad(i1) PW + k2]: the plane's half spectrum
    static __device__ __forceinline__ int at(int i1, int k2) { return lpad(i1) * PW + k2; }
};

// Forward axis-2 transforms of the plane's rows, the row's pairs given in v, to M.
template <int N>
__device__ __forceinline__ void plane_rows_r2c(float2 (&v)[Plane<N>::EX], float2* lds,
                                               const float2* __restrict__ tw, int twN,
                                               const float2* __restrict__ st) {
    using P = Plane<N>;
    constexpr int H = P::H;
    const int r = threadIdx.x / P::TX, j = threadIdx.x % P::TX;
    const bool act = r < N;
    float2* L = act ? lds + r * P::LS : lds + P::SLOTS + (r - N) % N * P::LS;
    fft_lds<H, P::EX, -1>(v, L, 1, 0, j, st);
    __syncthreads();
    float2 nyq = make_float2(0.f, 0.f);
#pragma unroll
    for (int e = 0; e < P::EX; ++e) {
        const int k = j + e * P::TX;
        float2 zk = L[lpad(k)], zc = cconj(L[lpad((H - k) & (H - 1))]);
        float2 A = cadd(zk, zc), B = csub(zk, zc);
        float2 w = tw[k * twN];
        float2 iwB = cmul_i<1>(cmul(w, B));
        float2 X = make_float2(0.5f * (A.x - iwB.x), 0.5f * (A.y - iwB.y));
        if (k == 0) {
            X = make_float2(zk.x + zk.y, 0.f);
            nyq = make_float2(zk.x - zk.y, 0.f);
        }
        v[e] = X;
    }
    __syncthreads();
    if (act) {
#pragma unroll
        for (int e = 0; e < P::EX; ++e) lds[P::at(r, j + e * P::TX)] = v[e];
        if (j == 0) lds[P::at(r, H)] = nyq;
    }
    __syncthreads();
}

// Axis-1 transforms of the plane's columns to M, in place for FROM_M, otherwise
// of value(i1, k2), all of whose loads are issued before the first transform.
template <int N, int DIR, bool FROM_M, class Value>
__device__ __forceinline__ void plane_columns(float2* lds, const float2* __restrict__ st,
                                              Value&& value) {
    using P = Plane<N>;
    const int j = threadIdx.x / P::PW, c = threadIdx.x % P::PW;
    const bool act = j < P::TY;
    float2 v[P::EY];
#pragma unroll
    for (int e = 0; e < P::EY; ++e) v[e] = value(act ? j + e * P::TY : 0, act ? c : 0);
    if constexpr (FROM_M) __syncthreads();   // M's columns are in registers
    fft_lds<N, P::EY, DIR>(v, act ? lds : lds + P::SLOTS, P::PW, c, act ? j : 0, st);
    __syncthreads();
}

// The plane's values i = p PW + k2 of M, NT at a time: f(round, p, k2, M value).
template <int N, class F>
__device__ __forceinline__ void plane_each(const float2* lds, F&& f) {
    using P = Plane<N>;
    constexpr int ALL = N * P::PW;
#pragma unroll
    for (int u = 0; u < (ALL + P::NT - 1) / P::NT; ++u) {
        const int i = u * P::NT + threadIdx.x;
        const int p = i / P::PW, k2 = i - p * P::PW;
        if (i < ALL) f(u, p, k2, lds[P::at(p, k2)]);
    }
}

// i k y with both products rounded (not contracted into the sums they enter), as
// in k_fft_x_c2r, which passes them through LDS.
__device__ __forceinline__ float2 times_ik(float k, float2 y) {
#pragma clang fp contract(off)
    return make_float2(-(k * y.y), k * y.x);
}

// Inverse axis-2 transforms of M's rows; the real rows' pairs end in lds, row r's
// pair k at lds[r LS + lpad(k)].  KMUL: times i k2 first (zero on the Nyquist
// column).
template <int N>
__device__ __forceinline__ void plane_rows_c2r(float2* lds, bool kmul,
                                               const float2 (&w)[Plane<N>::EX],
                                               const float2* __restrict__ st) {
    using P = Plane<N>;
    constexpr int H = P::H;
    const int r = threadIdx.x / P::TX, j = threadIdx.x % P::TX;
    const bool act = r < N;
    auto value = [&](int k) {
        const float2 y = lds[P::at(act ? r : 0, k)];
        if (!kmul) return y;
        if (k == H) return make_float2(0.f, 0.f);
        return times_ik((float)k, y);
    };
    float2 v[P::EX];
#pragma unroll
    for (int e = 0; e < P::EX; ++e) {
        const int k = j + e * P::TX;
        const float2 xk = value(k), xc = cconj(value(H - k));
        v[e] = cadd(cadd(xk, xc), cmul_i<1>(cmulc(csub(xk, xc), w[e])));
    }
    __syncthreads();
    float2* L = act ? lds + r * P::LS : lds + P::SLOTS + (r - N) % N * P::LS;
    fft_lds<H, P::EX, 1>(v, L, 1, 0, j, st);
    __syncthreads();
}

// Forward: real rows of plane blockIdx.x (in buffer blockIdx.y, or in the dense
// array `real` when given) -> half spectrum along axes 2 and 1 in the buffer.
// MERGE: buffer 0 like that; grid row 1 takes buffers 1 and 2 together and leaves
// n1 S_1 + k2 S_2 of their spectra in buffer 1 (as k_fft_y_merge).
template <int N, bool MERGE>
__global__ void __launch_bounds__(Plane<N>::NT)
k_plane_r2c(const float* __restrict__ real, float2* __restrict__ buf, int cs, long bufStride,
            const float2* __restrict__ tw, int ntw, const float2* __restrict__ st) {
    using P = Plane<N>;
    __shared__ float2 lds[P::ALL];
    const int i0 = (int)xcd_block(blockIdx.x, N), twN = ntw / N;
    const int r = threadIdx.x / P::TX, j = threadIdx.x % P::TX;
    const bool two = MERGE && blockIdx.y == 1;
    float2* b = buf + blockIdx.y * bufStride;
    auto load = [&](const float2* from, float2 (&v)[P::EX]) {
        const int i1 = r < N ? r : 0;
        const float* row = real ? real + ((long)i0 * N + i1) * N
                                : reinterpret_cast<const float*>(from + mesh_row(i0, i1, N) * cs);
#pragma unroll
        for (int e = 0; e < P::EX; ++e) {
            const int k = 2 * (j + e * P::TX);
            v[e] = make_float2(row[k], row[k + 1]);
        }
    };
    float2 v[P::EX], v2[P::EX];
    load(b, v);
    if (two) load(b + bufStride, v2);
    auto column = [&](int i1, int k2) { return lds[P::at(i1, k2)]; };
    plane_rows_r2c<N>(v, lds, tw, twN, st);
    plane_columns<N, -1, true>(lds, st, column);
    if (!two) {
        plane_each<N>(lds, [&](int, int p, int k2, float2 y) {
            b[mesh_row(i0, p, N) * cs + k2] = y;
        });
        return;
    }
    if constexpr (MERGE) {
        // n1 S_1, held by the thread that adds k2 S_2 to it
        float2 h[(N * P::PW + P::NT - 1) / P::NT];
        plane_each<N>(lds, [&](int u, int p, int, float2 y) {
            const float f1 = p == N / 2 ? 0.f : (float)signed_freq(p, N);
            h[u] = make_float2(f1 * y.x, f1 * y.y);
        });
        __syncthreads();   // the first spectrum has been read
        plane_rows_r2c<N>(v2, lds, tw, twN, st);
        plane_columns<N, -1, true>(lds, st, column);
        plane_each<N>(lds, [&](int u, int p, int k2, float2 y) {
            const float f2 = k2 == P::H ? 0.f : (float)k2;
            b[mesh_row(i0, p, N) * cs + k2] = make_float2(h[u].x + f2 * y.x, h[u].y + f2 * y.y);
        });
    }
}

// Inverse: spectrum of plane blockIdx.x -> real rows, in place in buffer
// blockIdx.y or to the dense array `real` when given (OPEN: unless *open is 0).  FORCE: grid row 0 takes
// buffer 0 in place; rows 1 and 2 both read `g` and leave the axis-1 derivative
// (times i n1 before the axis-1 transform) in buffer 1 and the axis-2 derivative
// (times i k2 before the axis-2 transform) in buffer 2.
template <int N, bool FORCE, bool OPEN>
__global__ void __launch_bounds__(Plane<N>::NT)
k_plane_c2r(float2* buf, const float2* __restrict__ g, float* __restrict__ real,
            const int* __restrict__ open, int cs, long bufStride, const float2* __restrict__ tw, int ntw,
            const float2* __restrict__ st) {
    using P = Plane<N>;
    __shared__ float2 lds[P::ALL];
    const int i0 = (int)xcd_block(blockIdx.x, N), comp = blockIdx.y;
    float2* b = buf + comp * bufStride;
    const float2* src = FORCE && comp > 0 ? g : b;
    const bool store = !OPEN || *open != 0;
    float2 w[P::EX];
#pragma unroll
    for (int e = 0; e < P::EX; ++e)
        w[e] = tw[(threadIdx.x % P::TX + e * P::TX) * (ntw / N)];
    auto spectrum = [&](int p, int k2) { return src[mesh_row(i0, p, N) * cs + k2]; };
    if (FORCE && comp == 1) {
        plane_columns<N, 1, false>(lds, st, [&](int p, int k2) {
            const float2 y = spectrum(p, k2);
            const float f1 = p == N / 2 ? 0.f : (float)signed_freq(p, N);
            return make_float2(-f1 * y.y, f1 * y.x);
        });
    } else {
        plane_columns<N, 1, false>(lds, st, spectrum);
    }
    plane_rows_c2r<N>(lds, FORCE && comp == 2, w, st);
    if (!store) return;
#pragma unroll
    for (int u = 0; u < (N * P::H + P::NT - 1) / P::NT; ++u) {
        const int i = u * P::NT + threadIdx.x;
        if (i >= N * P::H) break;
        const int p = i / P::H, k = i % P::H;
        float* row = real ? real + ((long)i0 * N + p) * N
                          : reinterpret_cast<float*>(b + mesh_row(i0, p, N) * cs);
        const float2 y = lds[p * P::LS + lpad(k)];
        row[2 * k] = y.x;
        row[2 * k + 1] = y.y;
    }
}

// Addresses of an axis-0 column's elements p = j + e T (mesh row (p, i1), column
// k2) of one lane.  Where T is a multiple of the row block's side, element e sits
// a wave-uniform e T H cs after element 0 (block and in-block indices are sums of
// separate i0 and i1 terms), and element 0 below 2^32 bytes.
template <int H>
struct Column {
    static constexpr int T = Cfg<H>::T;
    int i1, k2, j, cs;
    __device__ __forceinline__ Column(int i1_, int k2_, int j_, int cs_)
        : i1(i1_), k2(k2_), j(j_), cs(cs_) {}
    template <class F>
    __device__ __forceinline__ F* at(F* base, int e) const {
        if constexpr (T % 16 == 0) {
            using Byte = typename std::conditional<std::is_const<F>::value, const char, char>::type;
            const uint32_t lane = (uint32_t)(
                ((mesh_row(j, 0, H) + mesh_row(0, i1, H)) * cs + k2) * sizeof(float2));
            return reinterpret_cast<F*>(reinterpret_cast<Byte*>(base + (long)e * T * H * cs) + lane);
        } else {
            return base + mesh_row(j + e * T, i1, H) * cs + k2;
        }
    }
};

// Axis-0 pass with the fused gradient multiply (see launch_grad_z).  Writes
// F~_0 = IFFT_0(i n0 radial delta) and G = IFFT_0(radial delta); F~_1 and F~_2
// are i n1 G and i n2 G, and since n1 and n2 are constant along axis 0 those
// factors are applied by the later passes (k_fft_y_split multiplies by i n1
// before its axis-1 transform, the last-axis C2R by i k2), so this pass stores
// two spectra instead of three.
//
// From 256 points on, each lane looks up the radial multiplier of |n0| <= H/2
// only, with its column, and passes it to the lanes of n0 and -n0 through LDS (as
// k_grad_z_pipe), and the column is addressed by a wave-uniform part and 32 bits
// per lane: 72 VGPRs instead of 95 and 527 -> 505 us per 512^3 launch.  Occupancy
// is not what bounds it (four work-groups per CU without the sharing: 534 us),
// nor are streaming stores of use at this size (561 us; with streaming loads 611),
// and 16 columns per tile cost more (653 us, one work-group per CU).
template <int H>
__global__ void __launch_bounds__(Cfg<H>::T * Cfg<H>::W)
k_grad_z(const float2* __restrict__ src, float2* __restrict__ dst, float2* __restrict__ dst_g,
         int cs, int ncb, const float* __restrict__ radial, const float2* __restrict__ st) {
    constexpr int E = Cfg<H>::E, T = Cfg<H>::T, W = Cfg<H>::W, n = H;
    constexpr bool SHARE = H >= 256;
    constexpr int EQ = SHARE ? (H / 2) / T + 1 : 1;   // lookups: q = j + e T, and q = H/2
    // exchange buffer | the H-point part of the stage-twiddle table (read from
    // LDS rather than hoisted into registers, which hold the column)
    __shared__ float2 lds[lds_slots(H) * W + H];
    __shared__ float rq[SHARE ? (H / 2 + 1) * W : 1];   // the multipliers by q = |n0|
    float2* tab = lds + lds_slots(H) * W;
    // read first in the second stage, after the first stage's barrier
    for (int i = threadIdx.x; i < H - 1; i += T * W) tab[i] = st[H + i];
    const int c = threadIdx.x % W, j = threadIdx.x / W;
    const int tile = (int)xcd_block(blockIdx.x, gridDim.x);
    const int i1 = tile / ncb, cb = tile % ncb;
    const int k2 = cb * W + c;
    const Column<H> col(i1, k2, j, cs);
    const int n1 = signed_freq(i1, n);
    const bool in_half = k2 <= n / 2;
    [[maybe_unused]] float nr[EQ];
    if constexpr (SHARE) {
#pragma unroll
        for (int e = 0; e < EQ; ++e) {
            const int q = e < EQ - 1 ? j + e * T : n / 2;
            nr[e] = radial[in_half ? q * q + n1 * n1 + k2 * k2 : 0];
        }
    }
    float2 v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = *col.at(src, e);
    if constexpr (SHARE) {
#pragma unroll
        for (int e = 0; e < EQ - 1; ++e) rq[(j + e * T) * W + c] = in_half ? nr[e] : 0.f;
        // keeps the H/2 lookup with the others (as in k_grad_adj_z_pipe)
        __asm__ volatile("" ::"v"(nr[EQ - 1]));
        if (j == 0) rq[(n / 2) * W + c] = in_half ? nr[EQ - 1] : 0.f;
    }
    fft_lds_tab<H, E, -1>(v, lds, W, c, j, tab);
    __syncthreads();
    // radial * delta (kept: the F~_0 multiplier is n0 times it)
    float2 d[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int p = j + e * T;
        const int n0 = signed_freq(p, n);
        float rad;
        if constexpr (SHARE) rad = rq[(p <= n / 2 ? p : n - p) * W + c];
        else rad = in_half ? radial[n0 * n0 + n1 * n1 + k2 * k2] : 0.f;
        const float2 x = lds[lpad(p) * W + c];
        d[e] = make_float2(rad * x.x, rad * x.y);
        v[e] = d[e];
    }
    __syncthreads();
    fft_lds_tab<H, E, 1>(v, lds, W, c, j, tab);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) *col.at(dst_g, e) = lds[lpad(j + e * T) * W + c];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int n0 = signed_freq(j + e * T, n);
        const float f0 = n0 == -n / 2 ? 0.f : (float)n0;
        v[e] = make_float2(-d[e].y * f0, d[e].x * f0);
    }
    __syncthreads();
    fft_lds_tab<H, E, 1>(v, lds, W, c, j, tab);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) *col.at(dst, e) = lds[lpad(j + e * T) * W + c];
}

// k_grad_z for the largest transforms, whose register footprint allows one
// work-group per CU: a persistent loop over tiles in which the column and the
// radial multipliers of the next tile are loaded while the current one is
// transformed, so that the loads overlap the transforms instead of alternating
// with them.  Work-group b takes tiles lw, lw + nwg, ... with lw its
// XCD-contiguous index, so the work-groups of one XCD work on neighbouring
// column blocks at any time.
//
// Vector-memory operations of a wave complete in issue order, so a wait for a
// load also waits for every load and store issued before it.  The loop is
// arranged so that it waits only for the prefetched column and multipliers,
// issued a tile earlier, and never for loads issued just before the wait: the
// stage twiddles are read from an LDS copy, the radial multipliers come with
// the prefetch, and the prefetch is unconditional (the last tile reloads
// itself) so that every path into the loop header leaves the same operations
// in flight.
//
// The radial multiplier is a table lookup at |n|^2, which scatters a tile's
// lookups over the whole table (one cache line per lookup, nearly); modes n0
// and -n0 share it, so each lane looks up only |n0| = q <= H/2 and the values
// reach the lanes of both modes through LDS (rq), halving the lookups.  The
// column itself streams through once: non-temporal loads and stores keep it
// from evicting the table from L2.
template <int H>
__global__ void __launch_bounds__(Cfg<H>::T * Cfg<H>::W)
k_grad_z_pipe(const float2* __restrict__ src, float2* __restrict__ dst,
              float2* __restrict__ dst_g, int cs, int ncb, int ntiles,
              const float* __restrict__ radial, const float2* __restrict__ st) {
    constexpr int E = Cfg<H>::E, T = Cfg<H>::T, W = Cfg<H>::W, n = H;
    constexpr int LS = lds_slots(H) * W;
    // radial lookups per lane: q = j + e T for e < EQ - 1, and q = H/2
    constexpr int EQ = (H / 2) / T + 1;
    static_assert(T % 16 == 0, "rows j + e T must share their in-block index");
    static_assert((H / 2) % T == 0, "q = j + e T covers 0 .. H/2 - 1");
    // lds: the transforms' exchange buffer; keep (unpadded: each lane reads
    // back only its own slots): radial * delta_k of the column (held in LDS
    // rather than registers, which hold the next column); tab: the H-point
    // part of the stage-twiddle table (H - 1 entries); rq: the tile's radial
    // multipliers by q = |n0|
    __shared__ float2 lds[LS + H * W + H];
    __shared__ float rq[(H / 2 + 1) * W];
    float2* keep = lds + LS;
    float2* tab = keep + H * W;
    for (int i = threadIdx.x; i < H - 1; i += T * W) tab[i] = st[H + i];
    const int c = threadIdx.x % W, j = threadIdx.x / W;
    const int nwg = (int)gridDim.x;
    const int lw = (int)xcd_block(blockIdx.x, gridDim.x);
    // Element p = j + e T of the column of tile (i1, cb) sits at
    //   mesh_row(p, i1) cs + cb W + c = e T n cs + [mesh_row(j, 0) + mesh_row(0, i1)] cs + cb W + c
    // in the blocked order (block and in-block indices are sums of separate i0
    // and i1 terms, and T is a multiple of the block side): a wave-uniform part
    // e T n cs and a per-lane part below 2^32 bytes.
    const long estride = (long)T * n * cs;
    auto lane_off = [&](int tile) -> uint32_t {
        return (uint32_t)(((mesh_row(j, 0, n) + mesh_row(0, tile / ncb, n)) * cs +
                           (tile % ncb) * W + c) * sizeof(float2));
    };
    auto at = [](const float2* base, long e_off, uint32_t lane) -> const float2* {
        return reinterpret_cast<const float2*>(reinterpret_cast<const char*>(base + e_off) + lane);
    };
    // table index of this lane's e-th lookup for a tile (0 off the stored
    // half, whose multipliers are replaced by zero)
    auto rad_index = [&](int tile, int e) -> int {
        const int n1 = signed_freq(tile / ncb, n), k2 = (tile % ncb) * W + c;
        const int q = e < EQ - 1 ? j + e * T : n / 2;
        return k2 <= n / 2 ? q * q + n1 * n1 + k2 * k2 : 0;
    };
    if (lw >= ntiles) return;
    float2 nx[E];
    float nr[EQ];
    {
        const uint32_t lo = lane_off(lw);
#pragma unroll
        for (int e = 0; e < EQ; ++e) nr[e] = radial[rad_index(lw, e)];
#pragma unroll
        for (int e = 0; e < E; ++e) nx[e] = ld_nt(at(src, e * estride, lo));
    }
    // no loads in flight on entry to the loop (see above)
    __builtin_amdgcn_s_waitcnt(0);
    for (int tile = lw; tile < ntiles; tile += nwg) {
        const bool in_half = (tile % ncb) * W + c <= n / 2;
        const uint32_t lo = lane_off(tile);
        float2 v[E];
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] = nx[e];
        // rq is free: the previous tile read it before its last transforms
#pragma unroll
        for (int e = 0; e < EQ - 1; ++e) rq[(j + e * T) * W + c] = in_half ? nr[e] : 0.f;
        if (j == 0) rq[(n / 2) * W + c] = in_half ? nr[EQ - 1] : 0.f;
        {
            const int next = tile + nwg < ntiles ? tile + nwg : tile;
            const uint32_t ln = lane_off(next);
#pragma unroll
            for (int e = 0; e < EQ; ++e) nr[e] = radial[rad_index(next, e)];
#pragma unroll
            for (int e = 0; e < E; ++e) nx[e] = ld_nt(at(src, e * estride, ln));
        }
        fft_lds_tab<H, E, -1>(v, lds, W, c, j, tab);
        __syncthreads();
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int p = j + e * T;
            const float rad = rq[(p <= n / 2 ? p : n - p) * W + c];
            const float2 x = lds[lpad(p) * W + c];
            v[e] = make_float2(rad * x.x, rad * x.y);
            keep[p * W + c] = v[e];
        }
        __syncthreads();
        fft_lds_tab<H, E, 1>(v, lds, W, c, j, tab);
        __syncthreads();
#pragma unroll
        for (int e = 0; e < E; ++e)
            st_nt(const_cast<float2*>(at(dst_g, e * estride, lo)), lds[lpad(j + e * T) * W + c]);
        // F~_0 multiplier i n0 (zero on the Nyquist plane) on the kept column;
        // each lane reads back only the slots it wrote itself
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int p = j + e * T;
            const int n0 = signed_freq(p, n);
            const float f0 = n0 == -n / 2 ? 0.f : (float)n0;
            const float2 d = keep[p * W + c];
            v[e] = make_float2(-d.y * f0, d.x * f0);
        }
        __syncthreads();
        fft_lds_tab<H, E, 1>(v, lds, W, c, j, tab);
        __syncthreads();
#pragma unroll
        for (int e = 0; e < E; ++e)
            st_nt(const_cast<float2*>(at(dst, e * estride, lo)), lds[lpad(j + e * T) * W + c]);
        __syncthreads();   // the next tile's first transform reuses lds
    }
}

// Axis-0 pass of the transposed gradient operator (see launch_grad_adj_z).
// Sum_j conj(i n_j R) G_j = -i R (n0 G_0 + n1 G_1 + n2 G_2); n1 and n2 are fixed
// along the column, so n1 G_1 + n2 G_2 comes combined from the axis-1 pass
// (k_fft_y_merge) as the second input spectrum: three column FFTs per tile
// (four with the filter cotangent).
// FILT: the mode's term of dL/df(|n|^2), summed over +-n0, goes to
// modes[(|n0| n + i1) cs + k2], which k_filter_shells adds up by |n|^2.  Added to
// the table with global atomics instead (34 M of them on 197k words at 512^3,
// each served at the memory side), they were two thirds of this pass: 1.49 ms
// with them, 0.77 ms now and 0.13 ms for the sums (128^3: 40 us, now 15 + 16).
template <int H, bool FILT>
__global__ void __launch_bounds__(Cfg<H>::T * Cfg<H>::W)
k_grad_adj_z(const float2* __restrict__ src, long srcStride, float2* dst,
             const float2* dens, int cs, int ncb, const float* __restrict__ radial,
             float* __restrict__ modes, float fscale, const float2* __restrict__ st) {
    constexpr int E = Cfg<H>::E, T = Cfg<H>::T, W = Cfg<H>::W, n = H;
    // exchange buffer | the H-point part of the stage-twiddle table (read from
    // LDS rather than hoisted into registers, which hold the column)
    __shared__ float2 lds[lds_slots(H) * W + H];
    float2* tab = lds + lds_slots(H) * W;
    // read first in the second stage, after the first stage's barrier
    for (int i = threadIdx.x; i < H - 1; i += T * W) tab[i] = st[H + i];
    const int c = threadIdx.x % W, j = threadIdx.x / W;
    const int tile = (int)xcd_block(blockIdx.x, gridDim.x);
    const int i1 = tile / ncb, cb = tile % ncb;
    const int k2 = cb * W + c;
    // element p of the column (mesh row (p, i1), column k2)
    auto off = [&](int p) -> long { return mesh_row(p, i1, n) * cs + k2; };
    const int n1 = signed_freq(i1, n);
    const bool in_half = k2 <= n / 2;
    float2 v[E], a[E];
    // forward FFT of G_0, kept as n0 G_0 (zero on its Nyquist plane)
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = src[off(j + e * T)];
    fft_lds_tab<H, E, -1>(v, lds, W, c, j, tab);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int n0 = signed_freq(j + e * T, n);
        const float f0 = n0 == -n / 2 ? 0.f : (float)n0;
        const float2 g = lds[lpad(j + e * T) * W + c];
        a[e] = make_float2(f0 * g.x, f0 * g.y);
    }
    // forward FFT of n1 G_1 + n2 G_2 (the second input spectrum), added
    {
        const float2* u = src + srcStride;
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] = u[off(j + e * T)];
    }
    __syncthreads();
    fft_lds_tab<H, E, -1>(v, lds, W, c, j, tab);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const float2 g = lds[lpad(j + e * T) * W + c];
        a[e].x += g.x;
        a[e].y += g.y;
    }
    if constexpr (FILT) {
        // dL/df(|n|^2) += mult Re(conj(Sum_j n_j G_j) i fscale/|n|^2 dens_k)
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] = dens[off(j + e * T)];
        __syncthreads();
        fft_lds_tab<H, E, -1>(v, lds, W, c, j, tab);
        __syncthreads();
        // each lane turns its own elements' dens_k into their contribution (in
        // the same LDS slot), then the modes n0 and -n0, which share |n|^2, are
        // added
        const float mult = (k2 == 0 || k2 == n / 2) ? 1.f : 2.f;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int p = j + e * T;
            const int n0 = signed_freq(p, n);
            const int nsq = n0 * n0 + n1 * n1 + k2 * k2;
            const float2 dk = lds[lpad(p) * W + c];
            // Re(conj(a) * i dk) = a.y dk.x - a.x dk.y
            const float fs = nsq > 0 && in_half
                                 ? mult * (fscale / (float)nsq * (a[e].y * dk.x - a[e].x * dk.y))
                                 : 0.f;
            lds[lpad(p) * W + c] = make_float2(fs, 0.f);
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int p = j + e * T;
            if (p > n / 2) continue;
            float fs = lds[lpad(p) * W + c].x;
            if (p != 0 && p != n / 2) fs += lds[lpad(n - p) * W + c].x;
            modes[((long)p * n + i1) * cs + k2] = fs;
        }
    }
    // delta_bar_k = -i R (n0 G_0 + n1 G_1 + n2 G_2)
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int n0 = signed_freq(j + e * T, n);
        const float rad = in_half ? radial[n0 * n0 + n1 * n1 + k2 * k2] : 0.f;
        v[e] = make_float2(rad * a[e].y, -rad * a[e].x);
    }
    __syncthreads();
    fft_lds_tab<H, E, 1>(v, lds, W, c, j, tab);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) dst[off(j + e * T)] = lds[lpad(j + e * T) * W + c];
}

// Work-group (s, t): the sums over the modes of |n0| = t, t + kFilterSplits, ... of
// k_grad_adj_z's terms, by |n|^2 = q in the shell s width <= q < (s + 1) width, to
// part[t][q].  A column (|n0|, +-n1) meets a shell in one run of k2, found from two
// square roots, so every term is read once and added in LDS (FP64).  16 lanes
// share a column: at width 8 n a run is some 16 values, one or two 64-byte
// reads (one lane per column and shells of a 256th of the table, about one
// value per run, took 548 us at 512^3; this takes 125 us, 11 us at 128^3).
// Every entry is written: no clearing pass.
constexpr int kFilterSplits = 16, kFilterThreads = 512;
__global__ void __launch_bounds__(kFilterThreads)
k_filter_shells(const float* __restrict__ modes, int n, int cs, int width, int ntab,
                float* __restrict__ part) {
    extern __shared__ double acc[];   // [width]
    const int q0 = (int)blockIdx.x * width, q1 = q0 + width;
    for (int i = threadIdx.x; i < width; i += kFilterThreads) acc[i] = 0.0;
    __syncthreads();
    const int m = n / 2;
    // smallest k >= 0 with k^2 >= x
    auto root = [](int x) {
        if (x <= 0) return 0;
        int k = (int)sqrtf((float)x);
        while (k * k >= x) --k;
        while (k * k < x) ++k;
        return k;
    };
    const int lane = threadIdx.x & 15, group = threadIdx.x >> 4;
    for (int p = blockIdx.y; p <= m; p += kFilterSplits) {
        // the columns that meet the shell at some 0 <= k2 <= m
        const int i_end = min(root(q1 - p * p), m + 1);
        for (int i1 = root(q0 - m * m - p * p) + group; i1 < i_end; i1 += kFilterThreads / 16) {
            const int r2 = p * p + i1 * i1;
            const int k1 = min(root(q1 - r2), m + 1);
            const float* row = modes + ((long)p * n + i1) * cs;
            // -n1 sits in row n - i1; n1 = 0 and the Nyquist plane have no partner
            const bool paired = i1 > 0 && i1 < m;
            const float* other = paired ? modes + ((long)p * n + n - i1) * cs : row;
            for (int k = root(q0 - r2) + lane; k < k1; k += 16) {
                const float a = row[k], b = other[k];
                atomicAdd(&acc[r2 + k * k - q0], (double)(paired ? a + b : a));
            }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < width; i += kFilterThreads)
        if (q0 + i < ntab) part[(long)blockIdx.y * ntab + q0 + i] = (float)acc[i];
}

__global__ void __launch_bounds__(256)
k_filter_sum(const float* __restrict__ part, int ntab, float* __restrict__ fbar) {
    const int q = blockIdx.x * 256 + threadIdx.x;
    if (q >= ntab) return;
    float v[kFilterSplits];
#pragma unroll
    for (int t = 0; t < kFilterSplits; ++t) v[t] = part[(long)t * ntab + q];
    double s = 0.0;
#pragma unroll
    for (int t = 0; t < kFilterSplits; ++t) s += v[t];
    fbar[q] = (float)s;
}

// k_grad_adj_z (without the filter cotangent) for the largest transforms, as a
// persistent loop over tiles like k_grad_z_pipe: the tile's radial lookups and
// its G_0 and n1 G_1 + n2 G_2 columns are loaded at the top of the tile, and the
// sum n0 G_0 + n1 G_1 + n2 G_2 of the forward transforms is kept in LDS.  As in
// k_grad_z_pipe, each lane looks up the radial multipliers of |n0| <= H/2 only
// and shares them through LDS, and the columns stream with non-temporal loads
// and stores.
template <int H>
__global__ void __launch_bounds__(Cfg<H>::T * Cfg<H>::W)
k_grad_adj_z_pipe(const float2* __restrict__ src, long srcStride, float2* dst, int cs, int ncb,
                  int ntiles, const float* __restrict__ radial, const float2* __restrict__ st) {
    constexpr int E = Cfg<H>::E, T = Cfg<H>::T, W = Cfg<H>::W, n = H;
    constexpr int LS = lds_slots(H) * W;
    constexpr int EQ = (H / 2) / T + 1;   // radial lookups per lane (k_grad_z_pipe)
    static_assert(T % 16 == 0, "rows j + e T must share their in-block index");
    static_assert((H / 2) % T == 0, "q = j + e T covers 0 .. H/2 - 1");
    // exchange buffer | keep (unpadded, own slots only) | stage twiddles
    __shared__ float2 lds[LS + H * W + H];
    __shared__ float rq[(H / 2 + 1) * W];
    float2* keep = lds + LS;
    float2* twl = keep + H * W;
    const int c = threadIdx.x % W, j = threadIdx.x / W;
    for (int i = threadIdx.x; i < H - 1; i += T * W) twl[i] = st[H + i];
    const int nwg = (int)gridDim.x;
    const int lw = (int)xcd_block(blockIdx.x, gridDim.x);
    // wave-uniform row-block part e T n cs and a 32-bit lane part (k_grad_z_pipe)
    const long estride = (long)T * n * cs;
    auto lane_off = [&](int tile) -> uint32_t {
        return (uint32_t)(((mesh_row(j, 0, n) + mesh_row(0, tile / ncb, n)) * cs +
                           (tile % ncb) * W + c) * sizeof(float2));
    };
    auto at = [](const float2* base, long e_off, uint32_t lane) -> const float2* {
        return reinterpret_cast<const float2*>(reinterpret_cast<const char*>(base + e_off) + lane);
    };
    const float2* u = src + srcStride;   // n1 G_1 + n2 G_2
    for (int tile = lw; tile < ntiles; tile += nwg) {
        const int i1 = tile / ncb, k2 = (tile % ncb) * W + c;
        const uint32_t lo = lane_off(tile);
        const int n1 = signed_freq(i1, n);
        const bool in_half = k2 <= n / 2;
        float nr[EQ];
#pragma unroll
        for (int e = 0; e < EQ; ++e) {
            const int q = e < EQ - 1 ? j + e * T : n / 2;
            nr[e] = radial[in_half ? q * q + n1 * n1 + k2 * k2 : 0];
        }
        float2 v[E], y[E];
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] = ld_nt(at(src, e * estride, lo));
#pragma unroll
        for (int e = 0; e < E; ++e) y[e] = ld_nt(at(u, e * estride, lo));
        // rq is free: the previous tile read it before its last transform
#pragma unroll
        for (int e = 0; e < EQ - 1; ++e) rq[(j + e * T) * W + c] = in_half ? nr[e] : 0.f;
        // keeps the H/2 lookup here, issued with the others: sunk into the
        // branch below, its wait would also wait for the columns
        __asm__ volatile("" ::"v"(nr[EQ - 1]));
        if (j == 0) rq[(n / 2) * W + c] = in_half ? nr[EQ - 1] : 0.f;
        // forward FFT of G_0, kept as n0 G_0 (zero on its Nyquist plane)
        fft_lds_tab<H, E, -1>(v, lds, W, c, j, twl);
        __syncthreads();
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int p = j + e * T;
            const int n0 = signed_freq(p, n);
            const float f0 = n0 == -n / 2 ? 0.f : (float)n0;
            const float2 g = lds[lpad(p) * W + c];
            keep[p * W + c] = make_float2(f0 * g.x, f0 * g.y);
        }
        // forward FFT of n1 G_1 + n2 G_2, added to the kept column
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] = y[e];
        __syncthreads();
        fft_lds_tab<H, E, -1>(v, lds, W, c, j, twl);
        __syncthreads();
        // delta_bar_k = -i R (n0 G_0 + n1 G_1 + n2 G_2); each lane reads back only
        // the kept slots it wrote itself
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int p = j + e * T;
            const float rad = rq[(p <= n / 2 ? p : n - p) * W + c];
            const float2 g = lds[lpad(p) * W + c], k = keep[p * W + c];
            const float2 a = make_float2(k.x + g.x, k.y + g.y);
            v[e] = make_float2(rad * a.y, -rad * a.x);
        }
        __syncthreads();
        fft_lds_tab<H, E, 1>(v, lds, W, c, j, twl);
        __syncthreads();
#pragma unroll
        for (int e = 0; e < E; ++e)
            st_nt(const_cast<float2*>(at(dst, e * estride, lo)), lds[lpad(j + e * T) * W + c]);
        __syncthreads();   // the next tile's first transform reuses lds
    }
}

// Shell b = round(|n|) of integer |n|^2 = q: sqrt(q) + 1/2 >= b exactly when
// q >= b^2 - b + 1, so the single-precision guess is put right in integers.
__device__ __forceinline__ int shell_of(int q) {
    int b = (int)(sqrtf((float)q) + 0.5f);
    if (q < b * b - b + 1) --b;
    else if (q >= b * b + b + 1) ++b;
    return b;
}

// Slot of value i of work-group b's partial sums: the memory of the tile it
// starts with, in a buffer of the spectrum's layout (3 nbins <= 3 H values in
// a tile of H W >= 8 H slots of 8 bytes).
template <int H>
__device__ __forceinline__ long shell_slot(int b, int i, int cs, int ncb) {
    constexpr int W = Cfg<H>::W;
    return mesh_row(i / W, b / ncb, H) * cs + (b % ncb) * W + i % W;
}

// Last (axis-0) pass of a forward transform that only feeds shell sums: per
// shell b = 1..nbins {Sum w |d_k|^2, Sum w |n|, Sum w} in FP64, w the multiplicity
// of a half-spectrum mode.  The spectrum is neither written nor read back (a
// transform pass that stores it and a binning pass that reads it moved 3c more
// bytes than this one's c).
//
// FP64 LDS atomics run at about one lane per cycle and were what bounded the
// binning, so a lane first adds what shares a shell: modes n0 and -n0, and then a
// run of E/2 consecutive |n0|, along which the shell number never falls, in
// registers; one atomic per sum and shell change.  Work-groups take several
// tiles (two work-groups per CU) and leave their sums to k_shell_reduce, in the
// slots of their first tile (in `part`, which may be the buffer itself: nobody
// else reads that tile): FP64 atomics on one HBM word take turns of some 50 ns.
// 256^3: 56 us for the binning pass, after 34 us for the transform pass; now
// 47 us for both with the reduction (51 us with atomics on the totals).
template <int H>
__global__ void __launch_bounds__(Cfg<H>::T * Cfg<H>::W)
k_fft_shells(const float2* buf, float2* part, int cs, int ncb, int ntiles, int nbins,
             const float2* __restrict__ st) {
    constexpr int E = Cfg<H>::E, T = Cfg<H>::T, W = Cfg<H>::W, L = (H / 2) / T;
    static_assert(L * T == H / 2 && L >= 1, "each lane bins a run of L values of |n0|");
    __shared__ float2 lds[lds_slots(H) * W + H];
    extern __shared__ double sums[];   // [2 nbins] power and |n|, then [nbins] counts
    uint32_t* count = reinterpret_cast<uint32_t*>(sums + 2 * nbins);
    float2* tab = lds + lds_slots(H) * W;
    for (int i = threadIdx.x; i < H - 1; i += T * W) tab[i] = st[H + i];
    for (int i = threadIdx.x; i < nbins; i += T * W) {
        sums[2 * i] = sums[2 * i + 1] = 0.0;
        count[i] = 0u;
    }
    __syncthreads();
    const int c = threadIdx.x % W, j = threadIdx.x / W;
    for (int tile = (int)xcd_block(blockIdx.x, gridDim.x); tile < ntiles; tile += gridDim.x) {
        const int i1 = tile / ncb, k2 = (tile % ncb) * W + c;
        const int n1 = signed_freq(i1, H);
        float2 v[E];
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] = buf[mesh_row(j + e * T, i1, H) * cs + k2];
        fft_lds_tab<H, E, -1>(v, lds, W, c, j, tab);
        __syncthreads();
        if (k2 <= H / 2) {
            const uint32_t w = (k2 == 0 || k2 == H / 2) ? 1u : 2u;
            const int r2 = n1 * n1 + k2 * k2;
            int shell = 0;
            uint32_t n = 0;
            double power = 0.0, radius = 0.0;
            auto flush = [&]() {
                if (n == 0 || shell < 1 || shell > nbins) return;
                atomicAdd(&sums[2 * (shell - 1)], power);
                atomicAdd(&sums[2 * (shell - 1) + 1], radius);
                atomicAdd(&count[shell - 1], n);
            };
            const int last = j == T - 1 ? H / 2 : j * L + L - 1;   // n0 = H/2 has no lane of its own
            for (int p = j * L; p <= last; ++p) {
                const int q = p * p + r2, b = shell_of(q);
                if (b != shell) {
                    flush();
                    shell = b;
                    n = 0;
                    power = radius = 0.0;
                }
                const float2 d = lds[lpad(p) * W + c];
                double s = (double)d.x * d.x + (double)d.y * d.y;
                uint32_t m = w;
                if (p != 0 && p != H / 2) {
                    const float2 g = lds[lpad(H - p) * W + c];
                    s += (double)g.x * g.x + (double)g.y * g.y;
                    m += w;
                }
                power += w * s;
                radius += m * sqrt((double)q);
                n += m;
            }
            flush();
        }
        __syncthreads();   // the next tile's transform reuses lds
    }
    const int b = (int)xcd_block(blockIdx.x, gridDim.x);
    for (int i = threadIdx.x; i < 3 * nbins; i += T * W) {
        const int k = i / 3, q = i - 3 * k;
        const double x = q == 2 ? (double)count[k] : sums[2 * k + q];
        *reinterpret_cast<double*>(part + shell_slot<H>(b, i, cs, ncb)) = x;
    }
}

// bins[i] = the sum of the nparts work-groups' values i, 64 values per
// work-group: each of its 16 waves adds every 16th part, then wave 0 adds the
// waves' sums, in a fixed order.  (The parts themselves come from FP64 LDS atomics,
// whose order varies: shell sums, and the P(k) and loss formed from them, repeat to
// rounding, not bit for bit.)
template <int H>
__global__ void __launch_bounds__(1024)
k_shell_reduce(const float2* __restrict__ part, int cs, int ncb, int nparts, int nvals,
               double* __restrict__ bins) {
    __shared__ double red[16][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int i = blockIdx.x * 64 + lane, ic = i < nvals ? i : nvals - 1;
    auto at = [&](int b) {
        return *reinterpret_cast<const double*>(part + shell_slot<H>(b, ic, cs, ncb));
    };
    double s = 0.0;
    int b = w;
    for (; b + 7 * 16 < nparts; b += 8 * 16) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = at(b + 16 * u);
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; b < nparts; b += 16) s += at(b);
    red[w][lane] = s;
    __syncthreads();
    if (w == 0 && i < nvals) {
        double t = 0.0;
#pragma unroll
        for (int k = 0; k < 16; ++k) t += red[k][lane];
        bins[i] = t;
    }
}

// Axis-0 pass of a radial cotangent, in place: forward transform of a spectrum
// already transformed along axes 2 and 1, times table[b - 1] for the modes of
// shell b = 1..nbins (0 elsewhere), inverse transform.
template <int H>
__global__ void __launch_bounds__(Cfg<H>::T * Cfg<H>::W, Cfg<H>::MINW)
k_fft_shell_scale(float2* __restrict__ buf, int cs, int ncb, int nbins,
                  const float* __restrict__ table, const float2* __restrict__ st) {
    constexpr int E = Cfg<H>::E, T = Cfg<H>::T, W = Cfg<H>::W;
    __shared__ float2 lds[lds_slots(H) * W + H];
    float2* tab = lds + lds_slots(H) * W;
    // read first in the second stage, after the first stage's barrier
    for (int i = threadIdx.x; i < H - 1; i += T * W) tab[i] = st[H + i];
    const int c = threadIdx.x % W, j = threadIdx.x / W;
    const int tile = (int)xcd_block(blockIdx.x, gridDim.x);
    const int i1 = tile / ncb, k2 = (tile % ncb) * W + c;
    const int n1 = signed_freq(i1, H), r2 = n1 * n1 + k2 * k2;
    auto off = [&](int p) -> long { return mesh_row(p, i1, H) * cs + k2; };
    float2 v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = buf[off(j + e * T)];
    fft_lds_tab<H, E, -1>(v, lds, W, c, j, tab);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int p = j + e * T, n0 = signed_freq(p, H);
        const int b = shell_of(n0 * n0 + r2);
        const bool in = b >= 1 && b <= nbins && k2 <= H / 2;
        const float t = in ? table[in ? b - 1 : 0] : 0.f;
        const float2 d = lds[lpad(p) * W + c];
        v[e] = make_float2(t * d.x, t * d.y);
    }
    __syncthreads();
    fft_lds_tab<H, E, 1>(v, lds, W, c, j, tab);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) buf[off(j + e * T)] = lds[lpad(j + e * T) * W + c];
}

// Calls f(std::integral_constant<int, n>) for the supported power-of-two sizes:
// plane_switch up to kMaxPlane, pass_switch above, size_switch all.
template <class F>
void plane_switch(int n, F&& f) {
    switch (n) {
        case 8: f(std::integral_constant<int, 8>{}); break;
        case 16: f(std::integral_constant<int, 16>{}); break;
        case 32: f(std::integral_constant<int, 32>{}); break;
        case 64: f(std::integral_constant<int, 64>{}); break;
        default: break;
    }
}
template <class F>
void pass_switch(int n, F&& f) {
    switch (n) {
        case 128: f(std::integral_constant<int, 128>{}); break;
        case 256: f(std::integral_constant<int, 256>{}); break;
        case 512: f(std::integral_constant<int, 512>{}); break;
        case 1024: f(std::integral_constant<int, 1024>{}); break;
        default: break;
    }
}
template <class F>
void size_switch(int n, F&& f) {
    if (n <= kMaxPlane) plane_switch(n, f);
    else pass_switch(n, f);
}

// real == nullptr: in place
template <int N>
void x_r2c(const float* real, float2* buf, int cs, int nbuf, long bufStride, const Twiddles& tw,
           hipStream_t s) {
    constexpr int ROWS = Cfg<N / 2>::ROWS, T = Cfg<N / 2>::T;
    long nrows = (long)N * N;
    dim3 grid((unsigned)((nrows + ROWS - 1) / ROWS), nbuf);
    if (real)
        hipLaunchKernelGGL((k_fft_x_r2c<N, true>), grid, dim3(T * ROWS), 0, s, real, buf, cs, nrows,
                           bufStride, tw.w, tw.n, tw.stages);
    else
        hipLaunchKernelGGL((k_fft_x_r2c<N, false>), grid, dim3(T * ROWS), 0, s, nullptr, buf, cs,
                           nrows, bufStride, tw.w, tw.n, tw.stages);
}

template <int N>
void x_c2r(float2* buf, float* real, int cs, int nbuf, long bufStride, int kmul_buf,
           const Twiddles& tw, hipStream_t s, const int* open = nullptr) {
    constexpr int ROWS = Cfg<N / 2>::ROWS, T = Cfg<N / 2>::T;
    long nrows = (long)N * N;
    dim3 grid((unsigned)((nrows + ROWS - 1) / ROWS), nbuf);
    if (real && open)
        hipLaunchKernelGGL((k_fft_x_c2r<N, true, true>), grid, dim3(T * ROWS), 0, s, buf, real,
                           open, cs, nrows, bufStride, kmul_buf, tw.w, tw.n, tw.stages);
    else if (real)
        hipLaunchKernelGGL((k_fft_x_c2r<N, true, false>), grid, dim3(T * ROWS), 0, s, buf, real,
                           nullptr, cs, nrows, bufStride, kmul_buf, tw.w, tw.n, tw.stages);
    else
        hipLaunchKernelGGL((k_fft_x_c2r<N, false, false>), grid, dim3(T * ROWS), 0, s, buf, nullptr,
                           nullptr, cs, nrows, bufStride, kmul_buf, tw.w, tw.n, tw.stages);
}

template <int N, int DIR, int AXIS, bool SPEC, class Spec>
void strided(float2* buf, Spec spec, int cs, int nbuf, long bufStride, const Twiddles& tw,
             hipStream_t s) {
    constexpr int W = Cfg<N>::WS, T = Cfg<N>::T;
    int ncb = cs / W;
    hipLaunchKernelGGL((k_fft_strided<N, DIR, AXIS, SPEC>), dim3(N * ncb, nbuf), dim3(T * W), 0, s,
                       buf, spec, cs, ncb, bufStride, tw.stages);
}

}  // namespace

void launch_fft_x_r2c(float2* buf, int n, int cs, int nbuf, long bufStride, const Twiddles& tw, hipStream_t s) {
    pass_switch(n, [&](auto nn) {
        x_r2c<decltype(nn)::value>(nullptr, buf, cs, nbuf, bufStride, tw, s);
    });
}

void launch_fft_x_r2c_from(const float* real, float2* buf, int n, int cs, const Twiddles& tw,
                           hipStream_t s) {
    pass_switch(n, [&](auto nn) { x_r2c<decltype(nn)::value>(real, buf, cs, 1, 0, tw, s); });
}

void launch_fft_x_c2r(float2* buf, int n, int cs, int nbuf, long bufStride, const Twiddles& tw, hipStream_t s) {
    pass_switch(n, [&](auto nn) {
        x_c2r<decltype(nn)::value>(buf, nullptr, cs, nbuf, bufStride, -1, tw, s);
    });
}

void launch_fft_x_c2r_to(float2* buf, float* real, int n, int cs, const Twiddles& tw,
                         hipStream_t s, const int* open) {
    pass_switch(n, [&](auto nn) {
        x_c2r<decltype(nn)::value>(buf, real, cs, 1, 0, -1, tw, s, open);
    });
}

void launch_fft_x_c2r_dk2(float2* buf, int n, int cs, int nbuf, long bufStride, int kmul_buf,
                          const Twiddles& tw, hipStream_t s) {
    pass_switch(n, [&](auto nn) {
        x_c2r<decltype(nn)::value>(buf, nullptr, cs, nbuf, bufStride, kmul_buf, tw, s);
    });
}

void launch_fft_y_split(float2* g, float2* out_g, int n, int cs, const Twiddles& tw,
                        hipStream_t s) {
    pass_switch(n, [&](auto nn) {
        constexpr int N = decltype(nn)::value;
        constexpr int W = Cfg<N>::WY, T = Cfg<N>::T;
        const int ncb = cs / W;
        hipLaunchKernelGGL(k_fft_y_split<N>, dim3(N * ncb), dim3(T * W), 0, s, g, out_g, cs, ncb,
                           tw.stages);
    });
}

void launch_fft_y_merge(float2* g1, const float2* g2, int n, int cs, const Twiddles& tw,
                        hipStream_t s) {
    pass_switch(n, [&](auto nn) {
        constexpr int N = decltype(nn)::value;
        constexpr int W = Cfg<N>::WY, T = Cfg<N>::T;
        const int ncb = cs / W;
        hipLaunchKernelGGL(k_fft_y_merge<N>, dim3(N * ncb), dim3(T * W), 0, s, g1, g2, cs, ncb,
                           tw.stages);
    });
}

void launch_fft_y(float2* buf, int n, int cs, int dir, int nbuf, long bufStride,
                  const Twiddles& tw, hipStream_t s) {
    pass_switch(n, [&](auto nn) {
        constexpr int N = decltype(nn)::value;
        if (dir < 0) strided<N, -1, 1, false>(buf, nullptr, cs, nbuf, bufStride, tw, s);
        else strided<N, 1, 1, false>(buf, nullptr, cs, nbuf, bufStride, tw, s);
    });
}

void launch_grad_z(const float2* src, float2* dst, float2* dst_g, int n, int cs,
                   const float* radial, const Twiddles& tw, hipStream_t s) {
    size_switch(n, [&](auto nn) {
        constexpr int NN = decltype(nn)::value;
        constexpr int W = Cfg<NN>::W, T = Cfg<NN>::T;
        int ncb = cs / W;
        if constexpr (NN == 1024) {
            const int ntiles = NN * ncb;
            const int nwg = std::min(ntiles, device_cus());
            hipLaunchKernelGGL(k_grad_z_pipe<NN>, dim3(nwg), dim3(T * W), 0, s, src, dst,
                               dst_g, cs, ncb, ntiles, radial, tw.stages);
        } else {
            hipLaunchKernelGGL(k_grad_z<NN>, dim3(NN * ncb), dim3(T * W), 0, s, src, dst,
                               dst_g, cs, ncb, radial, tw.stages);
        }
    });
}

void launch_grad_adj_z(const float2* src, long srcStride, float2* dst, const float2* dens,
                       int n, int cs, const float* radial, float* fbar, float* modes,
                       float fscale, const Twiddles& tw, hipStream_t s) {
    size_switch(n, [&](auto nn) {
        constexpr int NN = decltype(nn)::value;
        constexpr int W = Cfg<NN>::W, T = Cfg<NN>::T;
        int ncb = cs / W;
        if (fbar) {
            hipLaunchKernelGGL((k_grad_adj_z<NN, true>), dim3(NN * ncb), dim3(T * W), 0, s, src,
                               srcStride, dst, dens, cs, ncb, radial, modes, fscale, tw.stages);
            constexpr int ntab = 3 * (NN / 2) * (NN / 2) + 1, width = 8 * NN;
            float* part = modes + (long)(NN / 2 + 1) * NN * cs;
            hipLaunchKernelGGL(k_filter_shells, dim3((ntab + width - 1) / width, kFilterSplits),
                               dim3(kFilterThreads), width * sizeof(double), s, modes, NN, cs,
                               width, ntab, part);
            hipLaunchKernelGGL(k_filter_sum, dim3((ntab + 255) / 256), dim3(256), 0, s, part, ntab,
                               fbar);
        } else if constexpr (NN == 1024) {
            const int ntiles = NN * ncb;
            const int nwg = std::min(ntiles, device_cus());
            hipLaunchKernelGGL(k_grad_adj_z_pipe<NN>, dim3(nwg), dim3(T * W), 0, s, src,
                               srcStride, dst, cs, ncb, ntiles, radial, tw.stages);
        } else {
            hipLaunchKernelGGL((k_grad_adj_z<NN, false>), dim3(NN * ncb), dim3(T * W), 0, s, src,
                               srcStride, dst, dens, cs, ncb, radial, nullptr, 0.f, tw.stages);
        }
    });
}

int device_cus() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus <= 0)
        return 256;
    return cus;
}

void fill_stage_twiddles(float2* table) {
    constexpr double kTwoPi = 6.283185307179586476925286766559;
    for (int i = 0; i < kStageTableSize; ++i) table[i] = make_float2(0.f, 0.f);
    for (int H = 2; H <= kMaxFft; H *= 2) {
        const int E = fft_values_per_lane(H);
        for (int Ns = 1; Ns < H;) {
            const int R = E < H / Ns ? E : H / Ns;
            if (Ns > 1)
                for (int r = 1; r < R; ++r)
                    for (int k = 0; k < Ns; ++k) {
                        const double ang = -kTwoPi * r * k / ((double)Ns * R);
                        table[H + (Ns - 1) + (r - 1) * Ns + k] =
                            make_float2((float)std::cos(ang), (float)std::sin(ang));
                    }
            Ns *= R;
        }
    }
}

void launch_fft_xy_r2c(const float* real, float2* buf, int n, int cs, int nbuf, long bufStride,
                       const Twiddles& tw, hipStream_t s) {
    if (n <= kMaxPlane) {
        plane_switch(n, [&](auto nn) {
            constexpr int N = decltype(nn)::value;
            hipLaunchKernelGGL((k_plane_r2c<N, false>), dim3(N, nbuf), dim3(Plane<N>::NT), 0, s,
                               real, buf, cs, bufStride, tw.w, tw.n, tw.stages);
        });
        return;
    }
    if (real) launch_fft_x_r2c_from(real, buf, n, cs, tw, s);
    else launch_fft_x_r2c(buf, n, cs, nbuf, bufStride, tw, s);
    launch_fft_y(buf, n, cs, -1, nbuf, bufStride, tw, s);
}

void launch_fft_yx_c2r(float2* buf, float* real, int n, int cs, int nbuf, long bufStride,
                       const Twiddles& tw, hipStream_t s, const int* open) {
    if (n <= kMaxPlane) {
        plane_switch(n, [&](auto nn) {
            constexpr int N = decltype(nn)::value;
            if (real && open)
                hipLaunchKernelGGL((k_plane_c2r<N, false, true>), dim3(N, nbuf),
                                   dim3(Plane<N>::NT), 0, s, buf, nullptr, real, open, cs,
                                   bufStride, tw.w, tw.n, tw.stages);
            else
                hipLaunchKernelGGL((k_plane_c2r<N, false, false>), dim3(N, nbuf),
                                   dim3(Plane<N>::NT), 0, s, buf, nullptr, real, nullptr, cs,
                                   bufStride, tw.w, tw.n, tw.stages);
        });
        return;
    }
    launch_fft_y(buf, n, cs, 1, nbuf, bufStride, tw, s);
    if (real) launch_fft_x_c2r_to(buf, real, n, cs, tw, s, open);
    else launch_fft_x_c2r(buf, n, cs, nbuf, bufStride, tw, s);
}

void launch_plane_r2c_merge(float2* buf, int n, int cs, long bufStride, const Twiddles& tw,
                            hipStream_t s) {
    plane_switch(n, [&](auto nn) {
        constexpr int N = decltype(nn)::value;
        hipLaunchKernelGGL((k_plane_r2c<N, true>), dim3(N, 2), dim3(Plane<N>::NT), 0, s, nullptr,
                           buf, cs, bufStride, tw.w, tw.n, tw.stages);
    });
}

void launch_plane_c2r_force(float2* buf, const float2* g, int n, int cs, long bufStride,
                            const Twiddles& tw, hipStream_t s) {
    plane_switch(n, [&](auto nn) {
        constexpr int N = decltype(nn)::value;
        hipLaunchKernelGGL((k_plane_c2r<N, true, false>), dim3(N, 3), dim3(Plane<N>::NT), 0, s, buf, g,
                           nullptr, nullptr, cs, bufStride, tw.w, tw.n, tw.stages);
    });
}

void launch_fft_z_mul(const float2* src, float2* dst, int n, int cs, int dir, int ax_a, int ax_b,
                      int mode, const float* table, float scale, bool accumulate,
                      const Twiddles& tw, hipStream_t s) {
    const LptMul M{ax_a, ax_b, mode, accumulate ? 1 : 0, table, scale};
    size_switch(n, [&](auto nn) {
        constexpr int N = decltype(nn)::value;
        constexpr int W = Cfg<N>::W, T = Cfg<N>::T;
        const int ncb = cs / W;
        if (dir > 0)
            hipLaunchKernelGGL((k_fft_z_mul<N, 1>), dim3(N * ncb), dim3(T * W), 0, s, src, dst, cs,
                               ncb, M, tw.stages);
        else
            hipLaunchKernelGGL((k_fft_z_mul<N, -1>), dim3(N * ncb), dim3(T * W), 0, s, src, dst, cs,
                               ncb, M, tw.stages);
    });
}

void launch_fft_shells(const float* real, float2* buf, float2* part, int n, int cs, int nbins,
                       double* bins, const Twiddles& tw, hipStream_t s) {
    launch_fft_xy_r2c(real, buf, n, cs, 1, 0, tw, s);
    size_switch(n, [&](auto nn) {
        constexpr int N = decltype(nn)::value;
        constexpr int W = Cfg<N>::W, T = Cfg<N>::T;
        const int ncb = (N / 2 + W) / W;   // column blocks that hold stored modes
        const int ntiles = N * ncb;
        const int nwg = std::min(ntiles, 2 * device_cus());
        hipLaunchKernelGGL(k_fft_shells<N>, dim3(nwg), dim3(T * W),
                           (2 * sizeof(double) + sizeof(uint32_t)) * nbins, s, buf, part, cs, ncb,
                           ntiles, nbins, tw.stages);
        hipLaunchKernelGGL(k_shell_reduce<N>, dim3((3 * nbins + 63) / 64), dim3(1024), 0, s, part,
                           cs, ncb, nwg, 3 * nbins, bins);
    });
}

void launch_fft_shell_scale(float2* buf, float* real, int n, int cs, int nbins, const float* table,
                            const int* open, const Twiddles& tw, hipStream_t s) {
    size_switch(n, [&](auto nn) {
        constexpr int N = decltype(nn)::value;
        constexpr int W = Cfg<N>::W, T = Cfg<N>::T;
        const int ncb = cs / W;
        hipLaunchKernelGGL(k_fft_shell_scale<N>, dim3(N * ncb), dim3(T * W), 0, s, buf, cs, ncb,
                           nbins, table, tw.stages);
    });
    launch_fft_yx_c2r(buf, real, n, cs, 1, 0, tw, s, open);
}

void launch_fft3_r2c_dense(const float* real, float2* buf, float2* spec, int n, int cs,
                           const Twiddles& tw, hipStream_t s) {
    launch_fft_xy_r2c(real, buf, n, cs, 1, 0, tw, s);
    size_switch(n, [&](auto nn) {
        constexpr int N = decltype(nn)::value;
        if (spec) strided<N, -1, 0, true>(buf, spec, cs, 1, 0, tw, s);
        else strided<N, -1, 0, false>(buf, nullptr, cs, 1, 0, tw, s);
    });
}

void launch_fft3_c2r_dense(const float2* spec, float2* buf, float* real, int n, int cs,
                           const Twiddles& tw, hipStream_t s) {
    size_switch(n, [&](auto nn) {
        constexpr int N = decltype(nn)::value;
        strided<N, 1, 0, true>(buf, spec, cs, 1, 0, tw, s);
    });
    launch_fft_yx_c2r(buf, real, n, cs, 1, 0, tw, s);
}

}  // namespace pmx
