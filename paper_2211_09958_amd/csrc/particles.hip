// Particle-side kernels for gfx950: cell-sorted bins, CIC scatter, CIC gather
// with the kick/drift update, and the adjoint (VJP) passes.
//
// Cloud-in-cell: a particle at u = x/cell - 1/2 (per axis) with i = floor(u),
// t = u - i gives weight (1 - t) to node i and t to node i + 1; the weight of a
// node is the product over the three axes.  Assignment (scatter) and
// interpolation (gather) use the same weights, so one is the transpose of the
// other; the weight's derivative is +-1/cell along the axis times the other two
// factors.
//
// State is fixed point (see kernels.h): positions are uint32 in units of
// box/2^32, so the base node is the top log2(ng) bits of x - cell/2 and t is
// read exactly from the low bits; momenta are int32.  The kick and drift add
// integer increments rounded from FP32 products by the shared helpers below,
// and the force is bitwise reproducible for a given state, so the reverse-time
// pass subtracts exactly what the forward pass added: the trajectory is
// recovered bit for bit.
//
// Bins: particles are counting-sorted by the T^3-cell tile holding their base
// node and by a 3-bit "spill class" (bit a set when the base node is on the
// last layer of the tile along axis a, i.e. the CIC footprint reaches the next
// tile).  The sort produces an order, ord[k] = storage slot of the k-th
// particle in bin order, rather than moving the records: particles move by a
// fraction of a cell per step, so the slots of one bin stay in a few long
// contiguous runs, and the records only need moving (compaction into bin
// order) every few sorts.  A work-group owns one tile: it accumulates its own
// particles and the spill classes of its 7 lower neighbours in LDS, then
// writes every cell of the tile exactly once -- no atomics to HBM, no
// pre-zeroing, coalesced rows.
// Densities accumulate as 64-bit fixed point (2^-32 units), so the result does
// not depend on the order of the LDS atomics (bitwise reproducible).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "kernels.h"
#include "layout.h"
#include "xcd.h"

namespace pmx {
namespace {

constexpr int kBlock = 256;
constexpr double kFix = 4294967296.0;  // 2^32

// Lattice coordinates of particle p (np a power of two: shifts and masks, since
// a 64-bit division takes some hundred instructions).
__device__ __forceinline__ void lattice_index(long p, int np, int jj[3]) {
    const int lg = __ffs(np) - 1, m = np - 1;
    jj[2] = (int)p & m;
    jj[1] = (int)(p >> lg) & m;
    jj[0] = (int)(p >> (2 * lg));
}

// Tiles are numbered in Morton (Z) order so that consecutive bins, and hence
// the work-groups resident on one XCD at a time, cover a compact 3-D block of
// the mesh.  Tiles per side is a power of two <= 256.
__device__ __forceinline__ uint32_t spread3(uint32_t v) {
    v &= 0xffu;
    v = (v | (v << 8)) & 0x0f00fu;
    v = (v | (v << 4)) & 0xc30c3u;
    v = (v | (v << 2)) & 0x249249u;
    return v;
}
__device__ __forceinline__ uint32_t compact3(uint32_t v) {
    v &= 0x249249u;
    v = (v | (v >> 2)) & 0xc30c3u;
    v = (v | (v >> 4)) & 0x0f00fu;
    v = (v | (v >> 8)) & 0xffu;
    return v;
}
__device__ __forceinline__ uint32_t morton3(uint32_t t0, uint32_t t1, uint32_t t2) {
    return (spread3(t0) << 2) | (spread3(t1) << 1) | spread3(t2);
}

// Base node index and fractional offset per axis from fixed-point positions.
__device__ __forceinline__ void locate(const uint32_t* __restrict__ x3, const Lattice& L, int ii[3],
                                       float t[3]) {
    const uint32_t mask = (1u << L.shift) - 1u;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const uint32_t u = x3[a] - L.half;
        ii[a] = (int)(u >> L.shift);
        t[a] = (float)(u & mask) * L.frac;
    }
}

// Momentum increment of a kick by coeff * F in integer units, before rounding.
__device__ __forceinline__ float kick_raw(float coeff, float F, const Lattice& L) {
    return __fmul_rn(__fmul_rn(coeff, F), L.inv_mom_unit);
}

// Integer momentum increment of a kick by coeff * F (forward adds, reverse subtracts).
__device__ __forceinline__ int32_t kick_units(float coeff, float F, const Lattice& L) {
    return __float2int_rn(kick_raw(coeff, F, L));
}

// Integer position increment of a drift by coeff * p, wrapped modulo the box.
__device__ __forceinline__ uint32_t drift_units(float coeff, int32_t pq, const Lattice& L) {
    const float d = __fmul_rn(__fmul_rn(coeff, __fmul_rn((float)pq, L.mom_unit)), L.len_to_pos);
    return (uint32_t)__float2ll_rn(d);
}

// Sum over a work-group of NTH threads; the total is valid in thread 0.
template <int NTH = kBlock>
__device__ __forceinline__ double block_sum(double v) {
    __shared__ double red[NTH / 64];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) red[wid] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < NTH / 64; ++w) s += red[w];
    __syncthreads();
    return s;
}

// Max over a work-group of NTH threads; valid in thread 0.
template <int NTH = kBlock>
__device__ __forceinline__ float block_max(float m) {
    __shared__ float red[NTH / 64];
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_down(m, o));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0)
        for (int w = 1; w < NTH / 64; ++w) m = fmaxf(m, red[w]);
    __syncthreads();
    return m;
}

// Max of a non-negative float over the block, as float bits atomically folded
// into *out by one lane per block (non-negative floats order like their bits).
__device__ __forceinline__ void block_max_to(float m, unsigned* out) {
    m = block_max(m);
    if (threadIdx.x == 0) atomicMax(out, __float_as_uint(m));
}

// ------------------------------------------------------------- binning

// Bin key of a particle at x: its tile (Morton number) times 8 plus its spill
// class.  tile is a power of two and the node indices are >= 0: shifts and
// masks instead of the (emulated) integer division and remainder by a
// run-time value.
__device__ __forceinline__ uint32_t bin_key(const uint32_t x[3], const Lattice& L, int tile) {
    int ii[3];
    float t[3];
    locate(x, L, ii, t);
    const int tl = __ffs(tile) - 1, tm = tile - 1;
    const uint32_t tix = morton3(ii[0] >> tl, ii[1] >> tl, ii[2] >> tl);
    const uint32_t cls = (((ii[0] & tm) == tm) << 2) | (((ii[1] & tm) == tm) << 1) |
                         ((ii[2] & tm) == tm);
    return tix * 8 + cls;
}

// Counts the particles of the active lanes into counts[key] and returns each
// one's rank among the particles of its key.  One atomic per distinct key in
// the wave, all issued together: the lanes are grouped by key first (no memory
// traffic), then every group's first lane adds the group size, and rank = that
// slot + the lane's place in its group.  Every active lane must call it.  The
// group's key is read with v_readlane (the leader is the same for all lanes):
// through the LDS crossbar, the loop waited for each of its up to 20 groups.
__device__ __forceinline__ uint32_t bin_rank(uint32_t key, uint32_t* __restrict__ counts) {
    const int lane = __lane_id();
    unsigned long long pending = __ballot(1);
    unsigned long long mine = 0ull;   // lanes sharing this lane's key
    while (pending) {   // all lanes of a key leave pending together
        const int leader = __ffsll((long long)pending) - 1;
        const uint32_t lk = (uint32_t)__builtin_amdgcn_readlane((int)key, leader);
        const unsigned long long same = __ballot(key == lk);
        if (key == lk) mine = same;
        pending &= ~same;
    }
    const int first = __ffsll((long long)mine) - 1;
    uint32_t base = 0;
    if (lane == first) base = atomicAdd(&counts[key], (uint32_t)__popcll(mine));
    base = (uint32_t)__shfl((int)base, first);
    return base + (uint32_t)__popcll(mine & ((1ull << lane) - 1ull));
}

__global__ void __launch_bounds__(kBlock)
k_bin_count(const uint32_t* __restrict__ xq, Lattice L, int tile, long P,
            uint32_t* __restrict__ counts, uint32_t* __restrict__ keys,
            uint32_t* __restrict__ ranks) {
    const long i = (long)xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
    if (i < P) {
        const uint32_t key = bin_key(xq + 3 * i, L, tile);
        const uint32_t rank = bin_rank(key, counts);
        keys[i] = key;
        ranks[i] = rank;
    }
}

// Particle i of the lattice in the order of the counting waves: a wave's 64 form a
// patch of 4 x 16 of a plane, and patches are numbered along the last axis first
// (plain lattice order below 16 particles per side).
__device__ __forceinline__ long patch_index(long i, int np, int jj[3]) {
    if (np < 16) {
        lattice_index(i, np, jj);
        return i;
    }
    const int lg = __ffs(np) - 1, lane = (int)i & 63;
    const long w = i >> 6;
    jj[2] = ((int)w & ((1 << (lg - 4)) - 1)) << 4 | (lane & 15);
    jj[1] = ((int)(w >> (lg - 4)) & ((1 << (lg - 2)) - 1)) << 2 | lane >> 4;
    jj[0] = (int)(w >> (2 * lg - 6));
    return (((long)jj[0] << lg | jj[1]) << lg) | jj[2];
}

// Displacements in lattice order -> fixed-point positions q + s, counted into
// the bins in the same pass (reading the positions back for the count would
// move as many bytes again).
//
// A wave takes a patch of 4 x 16 particles of a lattice plane (rows of 192 bytes):
// bin_rank takes a turn and an atomic per distinct bin in the wave, and a row of 64
// crosses four tiles or more.  512^3 particles on 512^3: 1375 -> 991 us (1.6 GB
// read, 2.7 GB written; 256^3 on 256^3: 190 -> 144); rows of 2 x 32 1110, 8 x 8 1343
// (96-byte rows), blocks of 2 x 2 x 16 1065, 4 x 4 x 4 1593.
__global__ void __launch_bounds__(kBlock)
k_to_fixed_count(const float* __restrict__ disp, uint32_t* __restrict__ xq, Lattice L, int tile,
                 long P, uint32_t* __restrict__ counts, uint32_t* __restrict__ keys,
                 uint32_t* __restrict__ ranks) {
    const long i = (long)xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
    if (i >= P) return;
    int jj[3];
    const long p = patch_index(i, L.np, jj);
    float d[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) d[a] = disp[3 * p + a];
    uint32_t x[3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
        x[a] = (uint32_t)jj[a] * L.qstep + (uint32_t)__float2ll_rn(__fmul_rn(d[a], L.len_to_pos));
#pragma unroll
    for (int a = 0; a < 3; ++a) xq[3 * p + a] = x[a];
    const uint32_t key = bin_key(x, L, tile);
    const uint32_t rank = bin_rank(key, counts);
    keys[i] = key;
    ranks[i] = rank;
}

// Exclusive block scan of 1024 threads x 4 values.
constexpr int kScanThreads = 1024, kScanPer = 4, kScanChunk = kScanThreads * kScanPer;

__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* total) {
    __shared__ uint32_t wsum[kScanThreads / 64];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    uint32_t incl = v;
    for (int o = 1; o < 64; o <<= 1) {
        uint32_t y = (uint32_t)__shfl_up((int)incl, o);
        if (lane >= o) incl += y;
    }
    if (lane == 63) wsum[wid] = incl;
    __syncthreads();
    if (wid == 0) {
        constexpr int NW = kScanThreads / 64;
        uint32_t w = lane < NW ? wsum[lane] : 0u;
        uint32_t wi = w;
        for (int o = 1; o < 64; o <<= 1) {
            uint32_t y = (uint32_t)__shfl_up((int)wi, o);
            if (lane >= o) wi += y;
        }
        if (lane < NW) wsum[lane] = wi - w;
        if (lane == NW - 1) *total = wi;
    }
    __syncthreads();
    uint32_t r = wsum[wid] + incl - v;
    __syncthreads();
    return r;
}

// Sum over the work-group, valid in every thread.
__device__ __forceinline__ uint32_t block_total(uint32_t v) {
    __shared__ uint32_t wsum[kScanThreads / 64];
    for (int o = 32; o > 0; o >>= 1) v += (uint32_t)__shfl_xor((int)v, o);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = v;
    __syncthreads();
    uint32_t t = 0;
#pragma unroll
    for (int w = 0; w < kScanThreads / 64; ++w) t += wsum[w];
    __syncthreads();
    return t;
}

// Exclusive scan of one chunk of kScanChunk values per work-group.  ONE: the
// whole scan in this launch, each work-group first adding up all the chunks
// before its own (for few chunks that costs less than two more launches);
// otherwise the chunk's total goes to bsum and k_scan_add finishes.
template <bool ONE>
__global__ void __launch_bounds__(kScanThreads)
k_scan_local(const uint32_t* __restrict__ in, uint32_t* __restrict__ out, long n,
             uint32_t* __restrict__ bsum) {
    __shared__ uint32_t tot;
    const long base = (long)blockIdx.x * kScanChunk + (long)threadIdx.x * kScanPer;
    uint32_t v[kScanPer], s = 0;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
        v[k] = base + k < n ? in[base + k] : 0u;
        s += v[k];
    }
    uint32_t before = 0;
    if constexpr (ONE) {
        const uint4* q = reinterpret_cast<const uint4*>(in);
        for (long i = threadIdx.x; i < (long)blockIdx.x * (kScanChunk / 4); i += kScanThreads) {
            const uint4 x = q[i];
            before += x.x + x.y + x.z + x.w;
        }
        before = block_total(before);
    }
    uint32_t ex = before + block_exclusive_scan(s, &tot);
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
        if (base + k < n) out[base + k] = ex;
        ex += v[k];
    }
    if (!ONE && threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// Adds the totals of the chunks before its own to every value of a chunk.
__global__ void __launch_bounds__(kScanThreads)
k_scan_add(uint32_t* __restrict__ out, long n, const uint32_t* __restrict__ bsum) {
    uint32_t add = 0;
    for (unsigned i = threadIdx.x; i < blockIdx.x; i += kScanThreads) add += bsum[i];
    add = block_total(add);
    const long base = (long)blockIdx.x * kScanChunk;
    for (int k = threadIdx.x; k < kScanChunk; k += kScanThreads)
        if (base + k < n) out[base + k] += add;
}

// Sorted order: the particle in storage slot i goes to bin position
// offsets[key] + rank.  keys and ranks are by slot, or, with np, in the order of
// the waves that counted a lattice set (patch_index), so that a wave's stores fall
// in few runs.  A chain of two loads and a store per particle: two particles per
// thread keep twice the loads in flight.  512^3 particles: 660 us with one, in slot
// order; 600 in patch order, 448 with two (four: 478), for 1.6 GB.  The bins' nk
// counts, read by the scan, are cleared for the next count.
constexpr int kIndexPer = 2;

__global__ void __launch_bounds__(kBlock)
k_index(const uint32_t* __restrict__ keys, const uint32_t* __restrict__ ranks,
        const uint32_t* __restrict__ offsets, long P, int np, uint32_t* __restrict__ ord,
        uint32_t* __restrict__ counts, long nk) {
    const long b0 = (long)xcd_block(blockIdx.x, gridDim.x) * (kBlock * kIndexPer) + threadIdx.x;
    uint32_t key[kIndexPer], rank[kIndexPer];
#pragma unroll
    for (int k = 0; k < kIndexPer; ++k) {
        const long i = b0 + k * kBlock;
        key[k] = i < P ? keys[i] : 0u;
        rank[k] = i < P ? ranks[i] : 0u;
    }
#pragma unroll
    for (int k = 0; k < kIndexPer; ++k) rank[k] += offsets[key[k]];
#pragma unroll
    for (int k = 0; k < kIndexPer; ++k) {
        const long i = b0 + k * kBlock;
        int jj[3];
        if (i < P) ord[rank[k]] = (uint32_t)(np ? patch_index(i, np, jj) : i);
    }
    const long i = (long)blockIdx.x * kBlock + threadIdx.x;
    if (i < nk) counts[i] = 0u;
}

// Scan and order in one launch for up to kScanChunk bins (meshes to 64^3): every
// work-group scans all the counts for itself, four per thread, and places 1024
// particles; the first one also stores the offsets.  Latency-bound: its loads are
// issued together, and what it costs is one launch where the scan and k_index
// took two (3.9 + 2.4 us at 32^3 particles on 64^3, now 4.2).  The counts, which
// all work-groups read, are cleared by the density scatter.
__global__ void __launch_bounds__(kScanThreads)
k_scan_index(const uint32_t* __restrict__ counts, uint32_t* __restrict__ offsets, int nk,
             const uint32_t* __restrict__ keys, const uint32_t* __restrict__ ranks, long P, int np,
             uint32_t* __restrict__ ord) {
    __shared__ uint32_t off[kScanChunk], tot;
    const long i = (long)xcd_block(blockIdx.x, gridDim.x) * kScanThreads + threadIdx.x;
    const uint32_t key = i < P ? keys[i] : 0u, rank = i < P ? ranks[i] : 0u;
    const int base = threadIdx.x * kScanPer;
    uint32_t v[kScanPer], s = 0;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
        v[k] = base + k < nk ? counts[base + k] : 0u;
        s += v[k];
    }
    uint32_t ex = block_exclusive_scan(s, &tot);
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
        off[base + k] = ex;
        if (blockIdx.x == 0 && base + k < nk) offsets[base + k] = ex;
        ex += v[k];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) offsets[nk] = tot;
    __syncthreads();
    int jj[3];
    if (i < P) ord[off[key] + rank] = (uint32_t)(np ? patch_index(i, np, jj) : i);
}

// Words per particle of the arrays of Records.
constexpr int kSortWords[5] = {3, 3, 1, 3, 3};

// Compaction of the first N of them: record k of every dst array
// <- record ord[k] of its src array, then ord[k] = k.  With the word counts
// fixed at compile time every gather load of a particle is issued before the
// first wait and before any store (a load after a store to an array the
// compiler cannot prove disjoint waits for the store; a branch on a run-time
// layout waits for the loads in it).
// LATTICE: as Records::lattice; a source that stands for zeros loads the position
// again instead, so that no load sits in a branch.
template <int N, bool LATTICE>
__global__ void __launch_bounds__(kBlock)
k_compact_sorted(uint32_t* __restrict__ ord, long P, Records rec) {
    const long k = (long)xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
    if (k >= P) return;
    const long i = ord[k];
    uint32_t buf[N][3];
#pragma unroll
    for (int a = 0; a < N; ++a) {
        if (LATTICE && a == 2) {
            buf[a][0] = (uint32_t)i;
            continue;
        }
        const bool zero = LATTICE && a > 2 && !rec.src[a];
        const uint32_t* src = (zero ? rec.src[0] : rec.src[a]) + i * kSortWords[a];
#pragma unroll
        for (int j = 0; j < kSortWords[a]; ++j) {
            const uint32_t v = src[j];
            buf[a][j] = zero ? 0u : v;
        }
    }
#pragma unroll
    for (int a = 0; a < N; ++a) {
        if (LATTICE && a == 4 && !rec.dst[a]) break;
        uint32_t* dst = rec.dst[a] + k * kSortWords[a];
#pragma unroll
        for (int j = 0; j < kSortWords[a]; ++j) dst[j] = buf[a][j];
    }
    ord[k] = (uint32_t)k;
}

// ------------------------------------------------------------- scatter

struct RangePairs {
    unsigned long long S = 0, cls = 0;
};
constexpr RangePairs range_pairs() {
    RangePairs p;
    int r = 0;
    for (unsigned long long S = 1; S < 8; ++S)
        for (unsigned long long cls = 0; cls < 8; ++cls)
            if ((cls & S) == S) {
                p.S |= S << (3 * r);
                p.cls |= cls << (3 * r);
                ++r;
            }
    return p;
}

// The 20 particle ranges a tile work-group visits: its own 8 classes, then for
// every non-empty axis subset S the classes of neighbour (tile - S) whose spill
// bits contain S.
__device__ __forceinline__ void tile_range(int r, int tx, int ty, int tz, int nt,
                                           const uint32_t* __restrict__ offsets,
                                           uint32_t* rs, uint32_t* re) {
    if (r == 0) {
        const uint32_t k0 = morton3(tx, ty, tz) * 8;
        *rs = offsets[k0];
        *re = offsets[k0 + 8];
        return;
    }
    // the (S, class) pairs with class containing S, three bits each
    constexpr RangePairs pairs = range_pairs();
    const int sh = 3 * (r - 1);
    const int S = (int)(pairs.S >> sh) & 7, cls = (int)(pairs.cls >> sh) & 7;
    const int m = nt - 1;   // nt is a power of two
    const uint32_t k = morton3((tx - ((S >> 2) & 1)) & m, (ty - ((S >> 1) & 1)) & m,
                               (tz - (S & 1)) & m) * 8 + cls;
    *rs = offsets[k];
    *re = offsets[k + 1];
}

constexpr int kRanges = 20;

// 64-bit fixed-point value of q (0 <= q < 2^62), rounded to nearest even: the
// same integer as rounding the exact (double) q, from single-precision
// operations only.  hi = floor(q / 2^32) is exact, and so is r = q - hi 2^32 in
// [0, 2^32): below 2^32 it is q itself, above it is a multiple of q's last place
// and at most 2^23 of those fit below 2^32; rounding r then rounds q.
__device__ __forceinline__ unsigned long long to_fixed64_nonneg(float q) {
    const float hi = floorf(q * 0x1p-32f);
    const float r = __builtin_rintf(__fmaf_rn(hi, -0x1p32f, q));
    return ((unsigned long long)(uint32_t)hi << 32) | (uint32_t)r;
}

// The same for |q| < 2^62 of either sign (two's complement); rounding to
// nearest even commutes with the sign.
__device__ __forceinline__ unsigned long long to_fixed64(float q) {
    const unsigned long long u = to_fixed64_nonneg(fabsf(q));
    return q < 0.f ? 0ull - u : u;
}

// LDS slot of tile cell (l0, l1, l2): row-major, with bits 2-3 of l2 swizzled
// by the row.  A 64-bit LDS word's bank pair depends on l2 alone in row-major
// order, and the lanes of a wave (particles consecutive in bin order, i.e.
// nearly in lattice order) share few l2 values across many rows; the swizzle
// spreads them over four bank groups.  It keeps groups of four consecutive
// cells together, so the write-out still reads them as two 16-byte words.
template <int T>
__device__ __forceinline__ int tile_slot(int l0, int l1, int l2) {
    constexpr int SW = T / 4 - 1;   // swizzle mask in units of four cells
    return (l0 * T + l1) * T + (l2 ^ (((l0 ^ l1) & SW) << 2));
}

// The 8 CIC corners of a particle at x that fall in the tile at lo, added to the
// tile's accumulator as the fixed-point value of w val 2^e, w the corner's
// weight (SIGNED: val may be negative).  Node
// indices and weights are formed once per axis; a corner outside the tile
// (the far node of a particle on the tile's last layer) is skipped.
template <int T, bool SIGNED>
__device__ __forceinline__ void deposit(unsigned long long* acc, const uint32_t x[3], float val,
                                        int e, const Lattice& L, const int lo[3]) {
    const int mask = L.ng - 1;
    int ii[3];
    float t[3];
    locate(x, L, ii, t);
    int l[3][2];
    bool in[3][2];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            int v = ((ii[a] + c) & mask) - lo[a];
            if (v < 0) v += L.ng;
            l[a][c] = v;
            in[a][c] = v < T;
        }
    }
#pragma unroll
    for (int c0 = 0; c0 < 2; ++c0) {
        if (!in[0][c0]) continue;
        const float w0 = c0 ? t[0] : 1.f - t[0];
#pragma unroll
        for (int c1 = 0; c1 < 2; ++c1) {
            if (!in[1][c1]) continue;
            const float w01 = w0 * (c1 ? t[1] : 1.f - t[1]);

#pragma unroll
            for (int c2 = 0; c2 < 2; ++c2) {
                if (!in[2][c2]) continue;
                const float w = w01 * (c2 ? t[2] : 1.f - t[2]);
                const float q = ldexpf(w * val, e);
                atomicAdd(&acc[tile_slot<T>(l[0][c0], l[1][c1], l[2][c2])],
                          SIGNED ? to_fixed64(q) : to_fixed64_nonneg(q));
            }
        }
    }
}

// The 8 CIC corners of a particle at x as LDS cells of the tile at lo and
// weights, with weight 0 for a corner outside the tile; cells packed two to a
// word (a tile has at most 2^12 cells).  Same arithmetic as deposit.
template <int T>
__device__ __forceinline__ void corners(const uint32_t x[3], const Lattice& L, const int lo[3],
                                        float w[8], uint32_t cell2[4]) {
    static_assert(T * T * T <= 4096, "cells are packed into 16 bits");
    const int mask = L.ng - 1;
    int ii[3];
    float t[3];
    locate(x, L, ii, t);
    int l[3][2];
    bool in[3][2];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            int v = ((ii[a] + c) & mask) - lo[a];
            if (v < 0) v += L.ng;
            l[a][c] = v;
            in[a][c] = v < T;
        }
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const int c0 = c >> 2, c1 = (c >> 1) & 1, c2 = c & 1;
        const float w01 = (c0 ? t[0] : 1.f - t[0]) * (c1 ? t[1] : 1.f - t[1]);
        const float wc = w01 * (c2 ? t[2] : 1.f - t[2]);
        w[c] = in[0][c0] && in[1][c1] && in[2][c2] ? wc : 0.f;
        const uint32_t cl = (uint32_t)tile_slot<T>(l[0][c0], l[1][c1], l[2][c2]) & 0xffffu;
        if (c & 1) cell2[c >> 1] |= cl << 16;
        else cell2[c >> 1] = cl;
    }
}

// deposit for corners kept by `corners` (a corner of weight 0 adds nothing).
__device__ __forceinline__ void deposit_kept(unsigned long long* acc, const float w[8],
                                             const uint32_t cell2[4], float val, int e) {
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        if (w[c] == 0.f) continue;
        const uint32_t cl = (c & 1) ? cell2[c >> 1] >> 16 : cell2[c >> 1] & 0xffffu;
        atomicAdd(&acc[cl], to_fixed64(ldexpf(w[c] * val, e)));
    }
}

// One work-group per tile.  Densities accumulate mass * w in 64-bit fixed
// point with 2^32 units; the vector scatter (VEC) accumulates coeff * v_j * w
// one component at a time, in 64-bit fixed point whose unit is chosen from
// max |coeff * v| and the particle count so that no sum can overflow.  Integer
// LDS atomics are both order-independent (bitwise reproducible results) and far
// faster on gfx950 than floating-point LDS atomics.  The kernel is bound by its
// vector-ALU instruction count (a wave64 instruction takes four cycles), so the
// per-corner work is kept to an index add, two products and the fixed-point
// conversion, and the write-out handles four cells per thread.  The density can
// also go to a caller's plain [ng]^3 array (dense), in the same write-out or
// instead of the workspace mesh (out null).
// Threads per scatter work-group; the 32 KB accumulator tile of T = 16 leaves
// room for four work-groups per CU, so larger ones keep more waves in flight.
// Smaller tiles hold an eighth of the particles, and the vector scatter
// accumulates its three components side by side instead of in three passes.
constexpr int scatter_threads(int T) { return T < 16 ? kBlock : 2 * kBlock; }

template <int T, bool VEC>
__global__ void __launch_bounds__(scatter_threads(T))
k_scatter_tile(const uint32_t* __restrict__ xq, const float* __restrict__ vals, float coeff,
               const unsigned* __restrict__ vmax_bits, Lattice L, int nt,
               const uint32_t* __restrict__ offsets, const uint32_t* __restrict__ ord,
               float* __restrict__ out, long outStride, float* __restrict__ dense,
               uint32_t* __restrict__ counts, int nk) {
    constexpr int T3 = T * T * T, NTH = scatter_threads(T);
    constexpr bool SIDE = VEC && T < 16;   // three accumulator tiles, one pass
    static_assert(T % 4 == 0, "the write-out handles four cells of a row at a time");
    __shared__ __align__(16) unsigned long long acc[SIDE ? 3 * T3 : T3];
    __shared__ uint32_t rs[kRanges], pre[kRanges + 1];
    const uint32_t tile = xcd_block(blockIdx.x, gridDim.x);
    const int tx = compact3(tile >> 2), ty = compact3(tile >> 1), tz = compact3(tile);
    const int lo[3] = {tx * T, ty * T, tz * T};
    if (!VEC && counts) {   // the bins' counts, read by k_scan_index (8 per tile)
        const int i = blockIdx.x * NTH + threadIdx.x;
        if (i < nk) counts[i] = 0u;
    }
    if (threadIdx.x < 64) {   // ranges and their prefix sum, in the first wave
        const int lane = threadIdx.x;
        uint32_t b = 0, e = 0;
        if (lane < kRanges) tile_range(lane, tx, ty, tz, nt, offsets, &b, &e);
        uint32_t incl = lane < kRanges ? e - b : 0u;
        for (int o = 1; o < 32; o <<= 1) {   // kRanges <= 32 lanes take part
            const uint32_t y = (uint32_t)__shfl_up((int)incl, o);
            if (lane >= o) incl += y;
        }
        if (lane < kRanges) {
            rs[lane] = b;
            pre[lane + 1] = incl;
        }
        if (lane == 0) pre[0] = 0u;
    }
    __syncthreads();
    int e = 32;
    double inv_scale = 1.0 / kFix;
    float amp = (float)(L.ratio * L.ratio * L.ratio);   // mass
    if constexpr (VEC) {
        // |Sum| <= P max|coeff v|: unit 2^-e with 2^e <= 2^62 / (P max|coeff v|)
        const double vmax = (double)fabsf(coeff) * (double)__uint_as_float(*vmax_bits);
        const double P = (double)L.np * L.np * L.np;
        e = 0;
        if (vmax > 0.0) {
            frexp(P * vmax, &e);
            e = 61 - e;
        }
        inv_scale = ldexp(1.0, -e);
        amp = coeff;
    }
    const uint32_t total = pre[kRanges];
    constexpr int NC = VEC ? 3 : 1;
    ulonglong2* acc2 = reinterpret_cast<ulonglong2*>(acc);
    float kw[8], kv[3];   // VEC: the kept first particle
    uint32_t kcell[4];
    // the accumulator starts at zero; each component's write-out clears the
    // slots it reads for the next one
    for (int c = threadIdx.x; c < (SIDE ? 3 : 1) * T3 / 2; c += NTH)
        acc2[c] = make_ulonglong2(0ull, 0ull);
    __syncthreads();
    // cell value v * 2^-e (minus the mean density 1 for the density), formed
    // from v's 32-bit halves with one rounding: hi 2^(32-e) + lo 2^-e exactly,
    // as the double conversion of v scaled by 2^-e (exact for |v| < 2^53, and
    // the same rounding of v beyond, since scaling by 2^-e commutes with it)
    const double hi_scale = inv_scale * 4294967296.0;
#pragma unroll
    for (int comp = 0; comp < NC; ++comp) {
        // one flat index space over the 20 ranges, so every lane has work.  A
        // particle's storage slot is loaded two iterations ahead and its record
        // one iteration ahead, so neither load is waited for before the atomics
        // of the particle in hand are issued
        // a thread looks up increasing indices (kk < total), so the range
        // search resumes where the previous lookup stopped
        int rcur = 0;
        auto slot = [&](uint32_t kk) {
            while (pre[rcur + 1] <= kk) ++rcur;
            return ord[rs[rcur] + (kk - pre[rcur])];
        };
        uint32_t nx[3] = {0u, 0u, 0u};
        float nv = 0.f;
        auto fetch = [&](uint32_t p) {
#pragma unroll
            for (int a = 0; a < 3; ++a) nx[a] = xq[3 * (long)p + a];
            if (VEC) nv = vals[3 * (long)p + comp];
        };
        uint32_t ns = 0;   // slot of the particle after the next
        uint32_t k = threadIdx.x;
        if constexpr (SIDE) {
            if (comp == 0) {
                uint32_t p = k < total ? slot(k) : 0u;
                for (; k < total; k += NTH) {
                    uint32_t x[3];
#pragma unroll
                    for (int a = 0; a < 3; ++a) x[a] = xq[3 * (long)p + a];
#pragma unroll
                    for (int a = 0; a < 3; ++a) kv[a] = vals[3 * (long)p + a];
                    if (k + NTH < total) p = slot(k + NTH);
                    corners<T>(x, L, lo, kw, kcell);
#pragma unroll
                    for (int a = 0; a < 3; ++a) deposit_kept(acc + a * T3, kw, kcell, amp * kv[a], e);
                }
            }
            k = total;   // nothing left for the passes below
        } else if constexpr (VEC) {
            // the thread's first particle: corners and values computed in the
            // first component's pass and kept for the other two
            if (comp == 0) {
                if (k < total) {
                    const uint32_t p = slot(k);
                    uint32_t x[3];
#pragma unroll
                    for (int a = 0; a < 3; ++a) x[a] = xq[3 * (long)p + a];
#pragma unroll
                    for (int c = 0; c < 3; ++c) kv[c] = vals[3 * (long)p + c];
                    corners<T>(x, L, lo, kw, kcell);
                }
            }
            if (k < total) deposit_kept(acc, kw, kcell, amp * kv[comp], e);
            k += NTH;
        }
        if (k < total) fetch(slot(k));
        if (k + NTH < total) ns = slot(k + NTH);
        for (; k < total; k += NTH) {
            const uint32_t cur[3] = {nx[0], nx[1], nx[2]};
            const float cv = nv;
            if (k + NTH < total) fetch(ns);
            if (k + 2 * NTH < total) ns = slot(k + 2 * NTH);
            deposit<T, VEC>(acc, cur, VEC ? amp * cv : amp, e, L, lo);   // densities are >= 0
        }
        __syncthreads();
        float* o = out + comp * outStride;
        for (int q = threadIdx.x; q < T3 / 4; q += NTH) {
            const int c = 4 * q;
            const int l2 = c % T, l1 = (c / T) % T, l0 = c / (T * T);
            const long g = mesh_row(lo[0] + l0, lo[1] + l1, L.ng) * L.rp + lo[2] + l2;
            const int sl = tile_slot<T>(l0, l1, l2) + (SIDE ? comp * T3 : 0);   // four in a row
            const ulonglong2 a = acc2[sl / 2], b = acc2[sl / 2 + 1];
            if (!SIDE && comp + 1 < NC) {
                acc2[sl / 2] = make_ulonglong2(0ull, 0ull);
                acc2[sl / 2 + 1] = make_ulonglong2(0ull, 0ull);
            }
            const unsigned long long v4[4] = {a.x, a.y, b.x, b.y};
            float r4[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                // the density's unit is 2^-32 (e = 32): minus 1 is minus 1 from hi
                const int hi = (int)(v4[i] >> 32) - (VEC ? 0 : 1);
                const unsigned lo = (unsigned)v4[i];
                r4[i] = (float)fma((double)lo, inv_scale, (double)hi * hi_scale);
            }
            if (VEC || out)
                *reinterpret_cast<float4*>(o + g) = make_float4(r4[0], r4[1], r4[2], r4[3]);
            if (!VEC && dense) {   // a caller's mesh: plain row order, any alignment
                float* d = dense + ((long)(lo[0] + l0) * L.ng + lo[1] + l1) * L.ng + lo[2] + l2;
                if ((reinterpret_cast<uintptr_t>(dense) & 15) == 0) {
                    *reinterpret_cast<float4*>(d) = make_float4(r4[0], r4[1], r4[2], r4[3]);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) d[i] = r4[i];
                }
            }
        }
        __syncthreads();
    }
}

// max |v| over n floats as float bits (non-negative floats order like their bits);
// 16-byte loads when v is 16-byte aligned (the maximum does not depend on the order).
// Every block ends in an atomic on the one result word, which take their turns
// (about 12 ns each): 1024 blocks with four loads in flight per thread instead
// of 4096 blocks with one, 50 -> 16.5 us for 128^3 particles (304 us, 5.3 TB/s, for 512^3).
__global__ void __launch_bounds__(kBlock)
k_absmax(const float* __restrict__ v, long n, unsigned* __restrict__ out) {
    float m = 0.f;
    const long first = (long)blockIdx.x * kBlock + threadIdx.x, stride = (long)gridDim.x * kBlock;
    long done = 0;
    if ((reinterpret_cast<uintptr_t>(v) & 15) == 0) {
        const float4* q = reinterpret_cast<const float4*>(v);
        done = 4 * (n / 4);
        auto max4 = [](float4 x) {
            return fmaxf(fmaxf(fabsf(x.x), fabsf(x.y)), fmaxf(fabsf(x.z), fabsf(x.w)));
        };
        long i = first;
        for (; i + 3 * stride < n / 4; i += 4 * stride) {
            const float4 x0 = q[i], x1 = q[i + stride], x2 = q[i + 2 * stride], x3 = q[i + 3 * stride];
            m = fmaxf(m, fmaxf(fmaxf(max4(x0), max4(x1)), fmaxf(max4(x2), max4(x3))));
        }
        for (; i < n / 4; i += stride) m = fmaxf(m, max4(q[i]));
    }
    for (long i = done + first; i < n; i += stride) m = fmaxf(m, fabsf(v[i]));
    block_max_to(m, out);
}

// ------------------------------------------------------------- gathers
//
// Gathers run one work-group per tile, like the scatter: the (T+1)^3 mesh
// values the tile's particles can touch are loaded into LDS with coalesced
// rows, then the particles of the tile's bin (through the sorted order)
// interpolate from LDS.  The interpolation uses explicitly rounded
// operations in a fixed order, so the forward gather and the reverse-time
// re-gather produce the same bits.

enum GatherMode { kKickDrift = 0, kForce = 1, kUnkickVjp = 2, kWgrad = 3 };

struct GatherArgs {
    uint32_t* xq;
    int32_t* pq;
    const uint32_t* id;   // kKickDrift checkpoints
    const float* mesh;    // 3 meshes mStride apart (1 for kWgrad)
    long mStride;
    long pitch;           // real-row pitch of the meshes
    int dense;            // 1: meshes in plain row order (a caller's [Ng]^3 array)
    float coeff;          // kick coefficient, or the mesh scale for kWgrad
    float drift;
    int flag;             // kKickDrift: drift?; kWgrad: 1 full reverse step, 2 xi only;
                          // kUnkickVjp: 1 xi starts at zero (not read)
    uint32_t* ck_x;       // kKickDrift checkpoint, lattice order (nullable)
    int32_t* ck_p;
    float* out;           // kForce output, by storage slot
    const float* pi_in;   // kUnkickVjp (null: zero, only p changes)
    float* xi;            // kUnkickVjp, kWgrad
    float* pi;            // kWgrad
    double* partials;     // one per tile (nullable)
    const uint32_t* ord;  // storage slot of each bin position
    // kKickDrift with drift, kWgrad flag 1: count the moved particles into the
    // next sort's bins (count != 0; pointers filled from the bins at launch)
    int count;
    uint32_t* bcounts;
    uint32_t* bkeys;
    uint32_t* branks;
    int btile;
    unsigned* ovf;        // kKickDrift: set to 1 when a momentum leaves the int32 range
    float* pmax;          // kWgrad flag 1: max |pi| written, one per tile (nullable)
};

// Threads per gather work-group: the three-mesh tile takes 59 KB of LDS (two
// work-groups per CU), so those modes use larger work-groups to keep more waves
// in flight.
constexpr int gather_threads(int mode, int T) {
    return mode == kWgrad || T < 16 ? kBlock : 4 * kBlock;
}

// A particle's inputs, loaded before any of its outputs is stored (a load after
// a store to an array that may alias it would wait a full memory round trip).
// Records are indexed in 64 bits (3 * (size_t)p + a): with a 32-bit index the
// compiler cannot rule out a wrap between a record's words and moves each word
// in an access of its own.
struct GatherRec {
    uint32_t x[3];
    int32_t pm[3];
    float xin[3], pin[3];
};

template <int MODE>
__device__ __forceinline__ void gather_load(const GatherArgs& A, uint32_t p, GatherRec& r) {
#pragma unroll
    for (int a = 0; a < 3; ++a) r.x[a] = A.xq[3 * (size_t)p + a];
    if constexpr (MODE == kKickDrift) {
#pragma unroll
        for (int a = 0; a < 3; ++a) r.pm[a] = A.pq[3 * (size_t)p + a];
    } else if constexpr (MODE == kUnkickVjp) {
        if (A.pq) {
#pragma unroll
            for (int a = 0; a < 3; ++a) r.pm[a] = A.pq[3 * (size_t)p + a];
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) r.pin[a] = r.xin[a] = 0.f;
        if (A.pi_in) {
#pragma unroll
            for (int a = 0; a < 3; ++a) r.pin[a] = A.pi_in[3 * (size_t)p + a];
            if (!A.flag) {
#pragma unroll
                for (int a = 0; a < 3; ++a) r.xin[a] = A.xi[3 * (size_t)p + a];
            }
        }
    } else if constexpr (MODE == kWgrad) {
#pragma unroll
        for (int a = 0; a < 3; ++a) r.xin[a] = A.xi[3 * (size_t)p + a];
        if (A.flag == 1) {
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                r.pm[a] = A.pq[3 * (size_t)p + a];
                r.pin[a] = A.pi[3 * (size_t)p + a];
            }
        }
    }
}

// The corners of a particle's cell in the tile at lo, whose meshes are in LDS.
template <int T, int NM>
struct TileMesh {
    static constexpr int TH = T + 1, TH3 = TH * TH * TH;
    const float* mf;
    const int* lo;
    int b[3];
    __device__ __forceinline__ void locate(const Lattice& L, const int ii[3]) {
#pragma unroll
        for (int a = 0; a < 3; ++a) b[a] = (ii[a] - lo[a]) & (L.ng - 1);   // in [0, T)
    }
    __device__ __forceinline__ float at(int m, int c0, int c1, int c2) const {
        return mf[m * TH3 + ((b[0] + c0) * TH + b[1] + c1) * TH + b[2] + c2];
    }
};

// The corners read from the meshes themselves, before anything else: a row's two
// nodes in one 8-byte load (in the last cell of a row, whose second node is the
// row's first, the pair before it and one more load).
template <int NM>
struct GlobalMesh {
    struct __attribute__((packed, aligned(4))) Pair {
        float a, b;
    };
    const GatherArgs& A;
    float f[NM][8];
    __device__ __forceinline__ void locate(const Lattice& L, const int ii[3]) {
        const int mask = L.ng - 1;
        const bool wrap = ii[2] == mask;
        const int i2 = wrap ? mask - 1 : ii[2];
        const float* row[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int r0 = (ii[0] + (r >> 1)) & mask, r1 = (ii[1] + (r & 1)) & mask;
            row[r] = A.mesh + (A.dense ? (long)r0 * L.ng + r1 : mesh_row(r0, r1, L.ng)) * A.pitch;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                const Pair v = *reinterpret_cast<const Pair*>(row[r] + m * A.mStride + i2);
                f[m][2 * r] = v.a;
                f[m][2 * r + 1] = v.b;
            }
        if (wrap) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int m = 0; m < NM; ++m) {
                    f[m][2 * r] = f[m][2 * r + 1];
                    f[m][2 * r + 1] = row[r][m * A.mStride];
                }
        }
    }
    __device__ __forceinline__ float at(int m, int c0, int c1, int c2) const {
        return f[m][4 * c0 + 2 * c1 + c2];
    }
};

// Interpolates the meshes at particle p and applies the mode's update; returns
// the particle's term of the mode's FP64 sum.
template <int MODE, class Mesh>
__device__ __forceinline__ double gather_apply(const GatherArgs& A, const Lattice& L, Mesh mesh,
                                               uint32_t p, const GatherRec& r, float& pmax) {
    constexpr int NM = MODE == kWgrad ? 1 : 3;
    const float ic = L.inv_cell;
    int ii[3];
    float t[3];
    locate(r.x, L, ii, t);
    mesh.locate(L, ii);
    // G[a]: the gradient of the interpolated mesh along axis a; for the
    // transposed kick only its contraction with the momentum cotangent is used,
    // Sum_m pin_m dF_m/dx_a = Sum_corners dw/dx_a (Sum_m pin_m f_m), which is
    // formed corner by corner (three accumulators instead of nine)
    float F[NM] = {0.f}, G[3] = {0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const int c0 = c >> 2, c1 = (c >> 1) & 1, c2 = c & 1;
        const float a0 = c0 ? t[0] : 1.f - t[0];
        const float a1 = c1 ? t[1] : 1.f - t[1];
        const float a2 = c2 ? t[2] : 1.f - t[2];
        const float w = __fmul_rn(__fmul_rn(a0, a1), a2);
        const float d0 = c0 ? ic : -ic, d1 = c1 ? ic : -ic, d2 = c2 ? ic : -ic;
        float g = 0.f;   // kWgrad: f; kUnkickVjp: Sum_m pin_m f_m
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            const float f = mesh.at(m, c0, c1, c2);
            if constexpr (MODE != kWgrad) F[m] = __fmaf_rn(w, f, F[m]);
            if constexpr (MODE == kUnkickVjp) g += r.pin[m] * f;
            if constexpr (MODE == kWgrad) g = f;
        }
        if constexpr (MODE == kUnkickVjp || MODE == kWgrad) {
            G[0] += d0 * a1 * a2 * g;
            G[1] += a0 * d1 * a2 * g;
            G[2] += a0 * a1 * d2 * g;
        }
    }
    double acc = 0.0;
    if constexpr (MODE == kKickDrift) {
        // p + increment in 64 bits: a sum or an increment outside the int32
        // range (or a non-finite force) would wrap silently, so it is flagged
        int32_t m[3];
        bool bad = false;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float q = kick_raw(A.coeff, F[a], L);
            const long long sum = (long long)r.pm[a] + __float2int_rn(q);
            m[a] = (int32_t)sum;
            bad = bad || !(fabsf(q) < 2.0e9f) || sum != (long long)m[a];
        }
        if (bad && A.ovf) atomicOr(A.ovf, 1u);
        // each array's three words stored together (one access each)
        if (A.ck_x) {
            const long q = A.id[p];
#pragma unroll
            for (int a = 0; a < 3; ++a) A.ck_x[3 * q + a] = r.x[a];
#pragma unroll
            for (int a = 0; a < 3; ++a) A.ck_p[3 * q + a] = m[a];
        }
        uint32_t xn[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) xn[a] = r.x[a] + drift_units(A.drift, m[a], L);
#pragma unroll
        for (int a = 0; a < 3; ++a) A.pq[3 * (size_t)p + a] = m[a];
        if (A.flag) {
#pragma unroll
            for (int a = 0; a < 3; ++a) A.xq[3 * (size_t)p + a] = xn[a];
        }
        if (A.flag && A.count) {
            const uint32_t key = bin_key(xn, L, A.btile);
            const uint32_t rank = bin_rank(key, A.bcounts);
            A.bkeys[p] = key;
            A.branks[p] = rank;
        }
    } else if constexpr (MODE == kForce) {
#pragma unroll
        for (int a = 0; a < 3; ++a) A.out[3 * (size_t)p + a] = F[a];
    } else if constexpr (MODE == kUnkickVjp) {
        if (A.pq) {
#pragma unroll
            for (int a = 0; a < 3; ++a) A.pq[3 * (size_t)p + a] = r.pm[a] - kick_units(A.coeff, F[a], L);
        }
        if (A.pi_in) {   // pi = 0 adds nothing to xi
#pragma unroll
            for (int a = 0; a < 3; ++a) A.xi[3 * (size_t)p + a] = r.xin[a] + A.coeff * G[a];
        }
        acc = (double)r.pin[0] * F[0] + (double)r.pin[1] * F[1] + (double)r.pin[2] * F[2];
    } else {   // kWgrad
        float xv[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            xv[a] = r.xin[a] + A.coeff * G[a];
            A.xi[3 * (size_t)p + a] = xv[a];
        }
        if (A.flag == 1) {
            uint32_t xn[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const int32_t m = r.pm[a];
                acc += (double)xv[a] * ((double)m * L.mom_unit);
                const float pn = r.pin[a] + A.drift * xv[a];
                A.pi[3 * (size_t)p + a] = pn;
                pmax = fmaxf(pmax, fabsf(pn));
                xn[a] = r.x[a] - drift_units(A.drift, m, L);
                A.xq[3 * (size_t)p + a] = xn[a];
            }
            if (A.count) {
                const uint32_t key = bin_key(xn, L, A.btile);
                const uint32_t rank = bin_rank(key, A.bcounts);
                A.bkeys[p] = key;
                A.branks[p] = rank;
            }
        }
    }
    return acc;
}

template <int T, int MODE>
__global__ void __launch_bounds__(gather_threads(MODE, T), MODE == kWgrad ? 1 : (T < 16 ? 4 : 8))
k_gather_tile(GatherArgs A, Lattice L, int nt, const uint32_t* __restrict__ offsets) {
    constexpr int NTH = gather_threads(MODE, T);
    constexpr int NM = MODE == kWgrad ? 1 : 3;
    constexpr int TH = T + 1, TH3 = TH * TH * TH;
    __shared__ float mf[NM * TH3];
    const uint32_t tile = xcd_block(blockIdx.x, gridDim.x);
    const int lo[3] = {(int)compact3(tile >> 2) * T, (int)compact3(tile >> 1) * T,
                       (int)compact3(tile) * T};
    const uint32_t pbeg = offsets[tile * 8], pend = offsets[tile * 8 + 8];
    const int mask = L.ng - 1;
    double acc = 0.0;
    float pmax = 0.f;
    if (pbeg < pend) {   // uniform across the work-group
        // this thread's first particle: its slot and inputs are loaded ahead of
        // the mesh tile, so their latency overlaps the tile's
        const uint32_t k0 = pbeg + threadIdx.x;
        uint32_t p0 = 0;
        GatherRec r0;
        if (k0 < pend) {
            p0 = A.ord[k0];
            gather_load<MODE>(A, p0, r0);
        }
        // the tile as NM (T+1)^2 columns along axis 0, one per thread: rows
        // i0 = lo0 .. lo0 + T - 1 lie a fixed number of storage rows apart (one
        // row-block side, or Ng in plain row order), so a column costs an
        // address add per value; row lo0 + T (which may wrap) is addressed apart
        const long step = (A.dense ? (long)L.ng : (1L << row_block_log2(L.ng))) * A.pitch;
        const int i0h = (lo[0] + T) & mask;
        for (int u = threadIdx.x; u < NM * TH * TH; u += NTH) {
            const int m = u / (TH * TH), pr = u - m * (TH * TH);
            const int l1 = pr / TH, l2 = pr - l1 * TH;
            const int i1 = (lo[1] + l1) & mask, i2 = (lo[2] + l2) & mask;
            const float* src = A.mesh + m * A.mStride + i2;
            const long row0 = A.dense ? (long)lo[0] * L.ng + i1 : mesh_row(lo[0], i1, L.ng);
            const long rowh = A.dense ? (long)i0h * L.ng + i1 : mesh_row(i0h, i1, L.ng);
            float* dst = mf + m * TH3 + pr;
            const float* col = src + row0 * A.pitch;
#pragma unroll
            for (int l0 = 0; l0 < T; ++l0) dst[l0 * TH * TH] = col[l0 * step];
            dst[T * TH * TH] = src[rowh * A.pitch];
        }
        __syncthreads();
        const TileMesh<T, NM> mesh{mf, lo};
        if (k0 < pend) acc += gather_apply<MODE>(A, L, mesh, p0, r0, pmax);
        for (uint32_t k = k0 + NTH; k < pend; k += NTH) {   // bins larger than the work-group
            const uint32_t p = A.ord[k];
            GatherRec r;
            gather_load<MODE>(A, p, r);
            acc += gather_apply<MODE>(A, L, mesh, p, r, pmax);
        }
    }
    if (A.partials) {
        const double s = block_sum<NTH>(acc);
        if (threadIdx.x == 0) A.partials[tile] = s;
    }
    if (MODE == kWgrad && A.pmax) {
        pmax = block_max<NTH>(pmax);
        if (threadIdx.x == 0) A.pmax[tile] = pmax;
    }
}

// The gathers for few particles per cell (gather_direct): the particles in storage
// order, each reading the nodes it needs from the meshes.  Where particles are
// cells apart, the tiles of k_gather_tile stage the whole meshes, mostly nodes
// that no particle reads, for 64 particles or fewer each; here the records stream
// and every line of mesh fetched is used by one or two particles.  Bound by the
// loads' latency and the lines they touch.
template <int MODE>
__global__ void __launch_bounds__(kBlock)
k_gather(GatherArgs A, Lattice L, long P, int per) {
    constexpr int NM = MODE == kWgrad ? 1 : 3;
    const long first = (long)xcd_block(blockIdx.x, gridDim.x) * per;
    double acc = 0.0;
    float pmax = 0.f;
    for (int c = 0; c < per; ++c) {
        const long p = (first + c) * kBlock + threadIdx.x;
        if (p >= P) break;
        GatherRec r;
        gather_load<MODE>(A, (uint32_t)p, r);
        acc += gather_apply<MODE>(A, L, GlobalMesh<NM>{A}, (uint32_t)p, r, pmax);
    }
    if (A.partials) {
        const double s = block_sum(acc);
        if (threadIdx.x == 0) A.partials[blockIdx.x] = s;
    }
    if (MODE == kWgrad && A.pmax) {
        pmax = block_max(pmax);
        if (threadIdx.x == 0) A.pmax[blockIdx.x] = pmax;
    }
}

// The particle part of a reverse step for a momentum cotangent that was zero:
// partials Sum xi . p, pi = drift xi, x -= drift p (exact inverse of the forward
// drift), the un-drifted particles counted into the next sort's bins.  Needs no
// mesh, so it streams the records in storage order.
__global__ void __launch_bounds__(kBlock)
k_undrift(uint32_t* __restrict__ xq, const int32_t* __restrict__ pq, const float* __restrict__ xi,
          float* __restrict__ pi, Lattice L, long P, float drift, int tile,
          uint32_t* __restrict__ counts, uint32_t* __restrict__ keys, uint32_t* __restrict__ ranks,
          double* __restrict__ partials, float* __restrict__ pmax) {
    double acc = 0.0;
    float mx = 0.f;
    for (long p = (long)xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x; p < P;
         p += (long)gridDim.x * kBlock) {
        uint32_t x[3];
        int32_t m[3];
        float v[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            x[a] = xq[3 * p + a];
            m[a] = pq[3 * p + a];
            v[a] = xi[3 * p + a];
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            acc += (double)v[a] * ((double)m[a] * L.mom_unit);
            x[a] -= drift_units(drift, m[a], L);
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) xq[3 * p + a] = x[a];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float pn = drift * v[a];
            pi[3 * p + a] = pn;
            mx = fmaxf(mx, fabsf(pn));
        }
        const uint32_t key = bin_key(x, L, tile);
        const uint32_t rank = bin_rank(key, counts);
        keys[p] = key;
        ranks[p] = rank;
    }
    const double s = block_sum(acc);
    mx = block_max(mx);
    if (threadIdx.x == 0) {
        partials[blockIdx.x] = s;
        pmax[blockIdx.x] = mx;
    }
}

// Final state of a forward run, to lattice order: displacement (minimum image of
// x - q) and momentum for the caller, and the fixed-point state for the adjoint.
__global__ void __launch_bounds__(kBlock)
k_final_state(const uint32_t* __restrict__ xq, const int32_t* __restrict__ pq,
              const uint32_t* __restrict__ id, Lattice L, long P, uint32_t* __restrict__ xo,
              int32_t* __restrict__ po, float* __restrict__ disp, float* __restrict__ mom) {
    const long p = (long)xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
    if (p >= P) return;
    const long q = id[p];
    uint32_t x[3];
    int32_t m[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) x[a] = xq[3 * p + a];
#pragma unroll
    for (int a = 0; a < 3; ++a) m[a] = pq[3 * p + a];
    int jj[3];
    lattice_index(q, L.np, jj);
#pragma unroll
    for (int a = 0; a < 3; ++a) xo[3 * q + a] = x[a];
#pragma unroll
    for (int a = 0; a < 3; ++a) po[3 * q + a] = m[a];
#pragma unroll
    for (int a = 0; a < 3; ++a)
        disp[3 * q + a] = (float)(int32_t)(x[a] - (uint32_t)jj[a] * L.qstep) * L.pos_to_len;
#pragma unroll
    for (int a = 0; a < 3; ++a) mom[3 * q + a] = (float)m[a] * L.mom_unit;
}

__global__ void __launch_bounds__(kBlock)
k_permute_by_id(const float* __restrict__ in, const uint32_t* __restrict__ id,
                float* __restrict__ out, long P) {
    for (long p = (long)xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x; p < P;
         p += (long)gridDim.x * kBlock) {
        const long q = id[p];
        float v[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) v[a] = in[3 * p + a];
#pragma unroll
        for (int a = 0; a < 3; ++a) out[3 * q + a] = v[a];
    }
}

__global__ void __launch_bounds__(kBlock) k_iota(uint32_t* __restrict__ id, long P) {
    for (long p = (long)xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x; p < P;
         p += (long)gridDim.x * kBlock)
        id[p] = (uint32_t)p;
}

// ------------------------------------------------------------- small kernels

// Work-group k: sums[slot[k]] = the sum of n[k] partials at src[k]; with maxs, one
// more work-group takes the maximum of nmax floats, as float bits, to *vmax.
__global__ void __launch_bounds__(1024)
k_reduce(ReduceSets R, double* __restrict__ sums) {
    __shared__ double red[16];
    if ((int)blockIdx.x == R.nsets) {
        float m = 0.f;
        for (int i = threadIdx.x; i < R.nmax; i += 1024) m = fmaxf(m, R.maxs[i]);
        m = block_max<1024>(m);
        if (threadIdx.x == 0) *R.vmax = __float_as_uint(m);
        return;
    }
    const double* partials = R.src[blockIdx.x];
    const int n = R.n[blockIdx.x];
    // four independent running sums per thread (a fixed order, so the result
    // repeats bit for bit), so that four loads are in flight instead of one
    double v0 = 0.0, v1 = 0.0, v2 = 0.0, v3 = 0.0;
    int i = threadIdx.x;
    for (; i + 3 * 1024 < n; i += 4 * 1024) {
        v0 += partials[i];
        v1 += partials[i + 1024];
        v2 += partials[i + 2 * 1024];
        v3 += partials[i + 3 * 1024];
    }
    for (; i < n; i += 1024) v0 += partials[i];
    double v = (v0 + v1) + (v2 + v3);
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < 16; ++w) s += red[w];
        sums[R.slot[blockIdx.x]] = s;
    }
}

// out (host memory mapped to the device): nsum sums, then nwords words and *last.
__global__ void __launch_bounds__(kBlock)
k_collect(const double* __restrict__ sums, int nsum, const unsigned* __restrict__ words, int nwords,
          const unsigned* __restrict__ last, double* __restrict__ out) {
    const int i = blockIdx.x * kBlock + threadIdx.x;
    unsigned* w = reinterpret_cast<unsigned*>(out + nsum);
    if (i < nsum) out[i] = sums[i];
    if (i < nwords) w[i] = words[i];
    if (i == nwords) w[i] = *last;
}

__global__ void __launch_bounds__(kBlock)
k_recon_err(const uint32_t* __restrict__ a, const uint32_t* __restrict__ id,
            const uint32_t* __restrict__ b, Lattice L, long P, double* partials,
            unsigned* maxbits) {
    double acc = 0.0;
    float mx = 0.f;
    for (long p = (long)xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x; p < P;
         p += (long)gridDim.x * kBlock) {
        const long q = id[p];
        float d2 = 0.f;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float d = (float)(int32_t)(a[3 * p + k] - b[3 * q + k]) * L.frac;
            d2 += d * d;
        }
        acc += d2;
        mx = fmaxf(mx, sqrtf(d2));
    }
    double s = block_sum(acc);
    if (threadIdx.x == 0) partials[blockIdx.x] = s;
    block_max_to(mx, maxbits);
}

// x = q + D0 s (+ D2 s2), p = G0 s (+ G2 s2) in fixed point for lattice
// particle p; s2 (the second-order field, 2LPT) is nullable.
__device__ __forceinline__ void ic_fixed(const float s[3], const float* s2, const int jj[3],
                                         float D0, float G0, float D2, float G2,
                                         const Lattice& L, uint32_t x[3], int32_t m[3]) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        float dx = __fmul_rn(D0, s[a]), dp = __fmul_rn(G0, s[a]);
        if (s2) {
            dx = __fmaf_rn(D2, s2[a], dx);
            dp = __fmaf_rn(G2, s2[a], dp);
        }
        x[a] = (uint32_t)jj[a] * L.qstep + (uint32_t)__float2ll_rn(__fmul_rn(dx, L.len_to_pos));
        m[a] = __float2int_rn(__fmul_rn(dp, L.inv_mom_unit));
    }
}

// s at the lattice site jj from three real meshes.
__device__ __forceinline__ void ic_field(const float* sm, long sStride, long o, float s[3]) {
#pragma unroll
    for (int a = 0; a < 3; ++a) s[a] = sm[a * sStride + o];
}

// What k_ic_state writes (lattice order): the fixed-point state and ids, that
// state as displacement and momentum, or s itself.
enum IcOutput { kIcFixed = 0, kIcFloat = 1, kIcField = 2 };

template <int OUT>
__global__ void __launch_bounds__(kBlock)
k_ic_state(const float* __restrict__ sm, long sStride, long rp, float D0, float G0, Lattice L,
           long P, uint32_t* __restrict__ xq, int32_t* __restrict__ pq, uint32_t* __restrict__ id,
           float* __restrict__ disp, float* __restrict__ mom, const float* __restrict__ s2v,
           float D2, float G2) {
    const long p = (long)xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
    if (p >= P) return;
    int jj[3];
    lattice_index(p, L.np, jj);
    float s[3], s2[3] = {0.f, 0.f, 0.f};
    ic_field(sm, sStride, mesh_row(jj[0], jj[1], L.np) * rp + jj[2], s);
    if constexpr (OUT == kIcField) {
#pragma unroll
        for (int a = 0; a < 3; ++a) disp[3 * p + a] = s[a];
        return;
    }
    if (s2v) {
#pragma unroll
        for (int a = 0; a < 3; ++a) s2[a] = s2v[3 * p + a];
    }
    uint32_t x[3];
    int32_t m[3];
    ic_fixed(s, s2v ? s2 : nullptr, jj, D0, G0, D2, G2, L, x, m);
    if constexpr (OUT == kIcFixed) {
#pragma unroll
        for (int a = 0; a < 3; ++a) xq[3 * p + a] = x[a];
#pragma unroll
        for (int a = 0; a < 3; ++a) pq[3 * p + a] = m[a];
        id[p] = (uint32_t)p;
    } else {
#pragma unroll
        for (int a = 0; a < 3; ++a)
            disp[3 * p + a] = (float)(int32_t)(x[a] - (uint32_t)jj[a] * L.qstep) * L.pos_to_len;
#pragma unroll
        for (int a = 0; a < 3; ++a) mom[3 * p + a] = (float)m[a] * L.mom_unit;
    }
}

// End of the adjoint, one pass over the particles (sorted order) where the
// check, six dot products and two weighted sums took one each: the
// reconstructed state against the ICs of lattice particle id[p], the cotangents
// against s and s2, and their combinations s_bar = D0 xi + G0 pi (over s in the
// meshes: a site is read and written by its own particle only) and s2_bar = D2 xi
// + G2 pi ([P][3], lattice order).  Block partials of kIcSums sums (see
// launch_ic_adjoint), the last three with LPT2 only.
template <bool LPT2>
__global__ void __launch_bounds__(kBlock)
k_ic_adjoint(float* sm, long sStride, long rp, float D0, float G0, Lattice L, long P,
             const uint32_t* __restrict__ xq, const int32_t* __restrict__ pq,
             const uint32_t* __restrict__ id, const float* __restrict__ xi,
             const float* __restrict__ pi, double* __restrict__ partials,
             unsigned* __restrict__ maxbits, const float* __restrict__ s2v,
             float* __restrict__ s2_bar, float D2, float G2) {
    constexpr int NS = LPT2 ? 9 : 6;
    double sum[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) sum[k] = 0.0;
    float mx = 0.f;
    for (long p = (long)xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x; p < P;
         p += (long)gridDim.x * kBlock) {
        const long lp = id[p];
        uint32_t xr[3];
        int32_t pr[3];
        float vx[3], vp[3], s[3], s2[3] = {0.f, 0.f, 0.f};
#pragma unroll
        for (int a = 0; a < 3; ++a) xr[a] = xq[3 * p + a];
#pragma unroll
        for (int a = 0; a < 3; ++a) pr[a] = pq[3 * p + a];
#pragma unroll
        for (int a = 0; a < 3; ++a) vx[a] = xi[3 * p + a];
#pragma unroll
        for (int a = 0; a < 3; ++a) vp[a] = pi[3 * p + a];
        int jj[3];
        lattice_index(lp, L.np, jj);
        const long o = mesh_row(jj[0], jj[1], L.np) * rp + jj[2];
        ic_field(sm, sStride, o, s);
        if constexpr (LPT2) {
#pragma unroll
            for (int a = 0; a < 3; ++a) s2[a] = s2v[3 * lp + a];
        }
        uint32_t x[3];
        int32_t m[3];
        ic_fixed(s, LPT2 ? s2 : nullptr, jj, D0, G0, D2, G2, L, x, m);
        float d2 = 0.f, b[3], b2[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float d = (float)(int32_t)(xr[a] - x[a]) * L.frac;
            d2 += d * d;
            const double dp = (double)pr[a] - m[a];
            sum[1] += dp * dp;
            sum[2] += (double)m[a] * m[a];
            b[a] = D0 * vx[a] + G0 * vp[a];
            sum[3] += (double)vx[a] * s[a];
            sum[4] += (double)vp[a] * s[a];
            sum[5] += (double)b[a] * s[a];
            sm[a * sStride + o] = b[a];
            if constexpr (LPT2) {
                b2[a] = D2 * vx[a] + G2 * vp[a];
                sum[6] += (double)vx[a] * s2[a];
                sum[7] += (double)vp[a] * s2[a];
                sum[8] += (double)b2[a] * s2[a];
            }
        }
        if constexpr (LPT2) {
#pragma unroll
            for (int a = 0; a < 3; ++a) s2_bar[3 * lp + a] = b2[a];
        }
        sum[0] += d2;
        mx = fmaxf(mx, sqrtf(d2));
    }
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        const double t = block_sum(sum[k]);
        if (threadIdx.x == 0) partials[(long)k * gridDim.x + blockIdx.x] = t;
    }
    block_max_to(mx, maxbits);
}

// ------------------------------------------------ 2LPT initial conditions

// Pointwise ops on real meshes of one layout (n^2 rows of pitch rp):
//   op 0  out = a b + a c + b c
//   op 1  out = a - b^2 (- c^2 when c is given)
//   op 2  out = scale a b
__global__ void __launch_bounds__(kBlock)
k_lpt_pointwise(const float* a, const float* b, const float* c, float* out, int n, long rp,
                int op, float scale) {
    const long N = (long)n * n * n;
    for (long i = (long)blockIdx.x * kBlock + threadIdx.x; i < N; i += (long)gridDim.x * kBlock) {
        const long o = (i / n) * rp + (i % n);
        const float x = a[o], y = b[o];
        float r;
        if (op == 0) {
            const float z = c[o];
            r = x * y + x * z + y * z;
        } else if (op == 1) {
            r = x - y * y;
            if (c) r -= c[o] * c[o];
        } else {
            r = scale * x * y;
        }
        out[o] = r;
    }
}

// dst[i] += scale * pitched src (compact [n]^3 dst).
__global__ void __launch_bounds__(kBlock)
k_add_from_pitched(const float* __restrict__ src, float* __restrict__ dst, int n, long rp,
                   float scale) {
    const long N = (long)n * n * n;
    for (long i = (long)blockIdx.x * kBlock + threadIdx.x; i < N; i += (long)gridDim.x * kBlock) {
        const long row = i / n;
        dst[i] += scale * src[mesh_row((int)(row / n), (int)(row % n), n) * rp + (i % n)];
    }
}

// Block partials of Sum_i pitched src_i * compact b_i.
__global__ void __launch_bounds__(kBlock)
k_dot_pitched(const float* __restrict__ src, const float* __restrict__ b, int n, long rp,
              double* partials) {
    const long N = (long)n * n * n;
    double acc = 0.0;
    for (long i = (long)blockIdx.x * kBlock + threadIdx.x; i < N; i += (long)gridDim.x * kBlock) {
        const long row = i / n;
        acc += (double)src[mesh_row((int)(row / n), (int)(row % n), n) * rp + (i % n)] * b[i];
    }
    double s = block_sum(acc);
    if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

__global__ void __launch_bounds__(kBlock)
k_deinterleave(const float* __restrict__ v, float* __restrict__ dst, long dstStride, int np, long rp) {
    const long P = (long)np * np * np;
    for (long p = (long)xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x; p < P;
         p += (long)gridDim.x * kBlock) {
        const long row = p / np;
        const long o = mesh_row((int)(row / np), (int)(row % np), np) * rp + (p % np);
#pragma unroll
        for (int a = 0; a < 3; ++a) dst[a * dstStride + o] = v[3 * p + a];
    }
}

__global__ void __launch_bounds__(kBlock)
k_mse(const float* __restrict__ d, const float* __restrict__ t, float* __restrict__ g, long n,
      float gscale, double* partials) {
    double acc = 0.0;
    for (long i = (long)blockIdx.x * kBlock + threadIdx.x; i < n; i += (long)gridDim.x * kBlock) {
        const float r = d[i] - t[i];
        acc += (double)r * r;
        if (g) g[i] = gscale * r;
    }
    double s = block_sum(acc);
    if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

// One work-group (see launch_pk_loss).
__global__ void __launch_bounds__(kBlock)
k_pk_loss(const double* __restrict__ bins, const double* __restrict__ target, int nbins,
          double norm, double weight, double* __restrict__ out, float* __restrict__ table,
          int* __restrict__ finite) {
    __shared__ double tot[2];
    double acc = 0.0, used = 0.0;
    auto usable = [&](int b) {
        return bins[3 * b + 2] > 0.0 && target[b] != 0.0 && isfinite(target[b]);
    };
    for (int b = threadIdx.x; b < nbins; b += kBlock)
        if (usable(b)) {
            const double r = bins[3 * b] / bins[3 * b + 2] * norm / target[b] - 1.0;
            acc += r * r;
            used += 1.0;
        }
    acc = block_sum(acc);
    used = block_sum(used);
    if (threadIdx.x == 0) {
        tot[0] = acc;
        tot[1] = used;
        out[0] = weight * acc / used;
        out[1] = acc;
        *finite = isfinite(acc) ? 1 : 0;
    }
    __syncthreads();
    for (int b = threadIdx.x; b < nbins; b += kBlock) {
        double t = 0.0;
        if (usable(b)) {
            const double r = bins[3 * b] / bins[3 * b + 2] * norm / target[b] - 1.0;
            t = 2.0 * (weight * 2.0 * r / (target[b] * tot[1])) * norm / bins[3 * b + 2];
        }
        table[b] = (float)t;
    }
}

// Periodic squared separation of two displacement arrays (minimum image, wrap
// d - box*floor(d/box + 1/2)); block partials of Sum d^2 and g = gscale * d.
__global__ void __launch_bounds__(kBlock)
k_mse_periodic(const float* __restrict__ a, const float* __restrict__ b, float* __restrict__ g,
               long n, float box, float inv_box, float gscale, double* partials) {
    double acc = 0.0;
    for (long i = (long)blockIdx.x * kBlock + threadIdx.x; i < n; i += (long)gridDim.x * kBlock) {
        float d = a[i] - b[i];
        d -= box * floorf(d * inv_box + 0.5f);
        acc += (double)d * d;
        if (g) g[i] = gscale * d;
    }
    double s = block_sum(acc);
    if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

__global__ void __launch_bounds__(kBlock) k_zero(uint32_t* __restrict__ p, long n) {
    for (long i = (long)blockIdx.x * kBlock + threadIdx.x; i < n; i += (long)gridDim.x * kBlock) p[i] = 0u;
}

// One thread per element: with XCD-aware numbering each XCD then sweeps one
// contiguous window of the (bin-sorted) particles.
int grid_for(long n) {
    long b = (n + kBlock - 1) / kBlock;
    return (int)(b < 1 ? 1 : b);
}

}  // namespace

// Tile side in cells.  Meshes up to 128^3 have at most 512 tiles of 16^3, too few
// for 256 CUs.  With 8^3 tiles the density scatter, the vector scatter and the
// kick, un-kick and mesh-gradient gathers of 32^3 particles on 64^3 take 5.7,
// 8.2, 6.0, 5.8 and 5.4 us instead of 6.8, 14.7, 8.7, 8.3 and 8.0; of 128^3
// particles on 128^3 19.4, 36, 34, 37 and 31 us instead of 19.4, 52, 28, 32 and
// 36 (the three-mesh gathers pay for the larger share of halo cells, about
// half of what the other two gain).  From 256^3 on, 16^3 tiles fill the chip, and
// their halos and key count are smaller.
int choose_tile(int ng) { return ng >= 256 ? 16 : (ng >= 16 ? 8 : 4); }

long scan_tmp_elems(long nkeys) { return (nkeys + 1 + kScanChunk - 1) / kScanChunk + 1; }

int particle_blocks(long P) {
    long b = (P + kBlock - 1) / kBlock;
    return (int)(b < 1 ? 1 : b);
}

void launch_zero(void* p, size_t bytes, hipStream_t s) {
    long n = (long)(bytes / 4);
    hipLaunchKernelGGL(k_zero, dim3(grid_for(n)), dim3(kBlock), 0, s, (uint32_t*)p, n);
}

// Whether one launch takes the scan and the order (k_scan_index).
static bool scan_with_order(const Bins& b) { return b.nkeys() <= kScanChunk; }

void launch_bin(const uint32_t* xq, const Lattice& L, Bins& b, Counted counted, hipStream_t s) {
    const long P = (long)L.np * L.np * L.np;
    const int np = counted == kCountedOnce ? L.np : 0;   // keys and ranks in patch order
    if (counted == kNotCounted) {
        launch_bin_zero(b, s);
        hipLaunchKernelGGL(k_bin_count, dim3((unsigned)((P + kBlock - 1) / kBlock)), dim3(kBlock), 0,
                           s, xq, L, b.tile, P, b.counts, b.keys, b.ranks);
    }
    if (scan_with_order(b)) {
        hipLaunchKernelGGL(k_scan_index, dim3((unsigned)((P + kScanThreads - 1) / kScanThreads)),
                           dim3(kScanThreads), 0, s, b.counts, b.offsets, (int)b.nkeys(), b.keys,
                           b.ranks, P, np, b.ord);
        return;
    }
    const long n = b.nkeys() + 1;
    const long nb = (n + kScanChunk - 1) / kScanChunk;
    // up to 16 chunks (meshes to 256^3) in one launch, about 3 us; the last of 16
    // work-groups then reads 240 KB more than its own chunk
    if (nb <= 16) {
        hipLaunchKernelGGL(k_scan_local<true>, dim3((unsigned)nb), dim3(kScanThreads), 0, s,
                           b.counts, b.offsets, n, b.scan_tmp);
    } else {
        hipLaunchKernelGGL(k_scan_local<false>, dim3((unsigned)nb), dim3(kScanThreads), 0, s,
                           b.counts, b.offsets, n, b.scan_tmp);
        hipLaunchKernelGGL(k_scan_add, dim3((unsigned)nb), dim3(kScanThreads), 0, s, b.offsets, n,
                           b.scan_tmp);
    }
    hipLaunchKernelGGL(k_index, dim3(grid_for(std::max((P + kIndexPer - 1) / kIndexPer, n))),
                       dim3(kBlock), 0, s, b.keys, b.ranks, b.offsets, P, np, b.ord, b.counts, n);
}

void launch_compact(Bins& b, const Records& rec, long P, hipStream_t s) {
    const dim3 grid((unsigned)((P + kBlock - 1) / kBlock));
    if (!rec.cotangents)
        hipLaunchKernelGGL((k_compact_sorted<3, false>), grid, dim3(kBlock), 0, s, b.ord, P, rec);
    else if (rec.lattice)
        hipLaunchKernelGGL((k_compact_sorted<5, true>), grid, dim3(kBlock), 0, s, b.ord, P, rec);
    else
        hipLaunchKernelGGL((k_compact_sorted<5, false>), grid, dim3(kBlock), 0, s, b.ord, P, rec);
}

template <bool VEC>
static void scatter_dispatch(const uint32_t* xq, const float* v, float coeff, const unsigned* vmax,
                             const Lattice& L, const Bins& b, float* out, long outStride,
                             float* dense, uint32_t* counts, hipStream_t s) {
    const int nk = (int)b.nkeys();
    const unsigned ntiles = (unsigned)b.nt * b.nt * b.nt;
    switch (b.tile) {
        case 4:
            hipLaunchKernelGGL((k_scatter_tile<4, VEC>), dim3(ntiles), dim3(scatter_threads(4)), 0, s, xq, v,
                               coeff, vmax, L, b.nt, b.offsets, b.ord, out, outStride, dense, counts, nk);
            break;
        case 8:
            hipLaunchKernelGGL((k_scatter_tile<8, VEC>), dim3(ntiles), dim3(scatter_threads(8)), 0, s, xq, v,
                               coeff, vmax, L, b.nt, b.offsets, b.ord, out, outStride, dense, counts, nk);
            break;
        default:
            hipLaunchKernelGGL((k_scatter_tile<16, VEC>), dim3(ntiles), dim3(scatter_threads(16)), 0, s, xq, v,
                               coeff, vmax, L, b.nt, b.offsets, b.ord, out, outStride, dense, counts, nk);
            break;
    }
}

void launch_scatter_density(const uint32_t* xq, const Lattice& L, const Bins& b, float* mesh,
                            float* dense, hipStream_t s) {
    scatter_dispatch<false>(xq, nullptr, 0.f, nullptr, L, b, mesh, 0, dense,
                            scan_with_order(b) ? b.counts : nullptr, s);
}

void launch_absmax(const float* v, long n, unsigned* out, hipStream_t s) {
    const long nb = std::min<long>(grid_for(n), 1024);
    hipLaunchKernelGGL(k_absmax, dim3((unsigned)nb), dim3(kBlock), 0, s, v, n, out);
}

void launch_scatter_vec(const uint32_t* xq, const float* v, float coeff, const unsigned* vmax,
                        const Lattice& L, const Bins& b, float* out, long outStride,
                        hipStream_t s) {
    scatter_dispatch<true>(xq, v, coeff, vmax, L, b, out, outStride, nullptr, nullptr, s);
}

// Particles at least four cells apart on a mesh of 128^3 or more: the nodes of
// their cells straight from the meshes (k_gather) instead of tiles of the meshes in
// LDS (128^3 particles on 512^3: transposed kick 596 -> 471 us, cotangent gather
// 217 -> 150; two steps and their adjoint 28.2 -> 25.7 ms, 256^3 on 1024^3 one step
// 161 -> 148 ms, five steps of 16^3 on 128^3 1.64 -> 1.61 ms).  At two cells the
// tiles are the faster ones (256^3 on 512^3: kick and drift 700 us against 930,
// transposed kick 765 against 956), at one cell by far (512^3 on 512^3: 2.2 ms
// against 7.3): neighbouring particles then share most of their lines.  Smaller
// meshes have too few particles for the grid (five steps of 16^3 on 64^3: 774 us
// against 808).
static bool gather_direct(int np, int ng) { return 4 * np <= ng && ng >= 128; }
struct GatherGrid {
    unsigned blocks;
    int per;   // chunks of kBlock particles per work-group
};
static GatherGrid gather_grid(long P) {
    const long chunks = (P + kBlock - 1) / kBlock, per = (chunks + 8191) / 8192;
    return {(unsigned)((chunks + per - 1) / per), (int)per};
}

template <int MODE>
static void gather_dispatch(GatherArgs A, const Lattice& L, const Bins& b, hipStream_t s) {
    const unsigned ntiles = (unsigned)b.nt * b.nt * b.nt;
    A.ord = b.ord;
    if (A.count) {   // the bins are read (ord, offsets) before the counts are reused
        A.bcounts = b.counts;
        A.bkeys = b.keys;
        A.branks = b.ranks;
        A.btile = b.tile;
    }
    if (gather_direct(L.np, L.ng)) {
        const long P = (long)L.np * L.np * L.np;
        const GatherGrid g = gather_grid(P);
        hipLaunchKernelGGL((k_gather<MODE>), dim3(g.blocks), dim3(kBlock), 0, s, A, L, P, g.per);
        return;
    }
    switch (b.tile) {
        case 4:
            hipLaunchKernelGGL((k_gather_tile<4, MODE>), dim3(ntiles), dim3(gather_threads(MODE, 4)), 0, s, A, L, b.nt,
                               b.offsets);
            break;
        case 8:
            hipLaunchKernelGGL((k_gather_tile<8, MODE>), dim3(ntiles), dim3(gather_threads(MODE, 8)), 0, s, A, L, b.nt,
                               b.offsets);
            break;
        default:
            hipLaunchKernelGGL((k_gather_tile<16, MODE>), dim3(ntiles), dim3(gather_threads(MODE, 16)), 0, s, A, L,
                               b.nt, b.offsets);
            break;
    }
}

long gather_partials(int np, int ng) {
    const long nt = ng / choose_tile(ng);
    return gather_direct(np, ng) ? gather_grid((long)np * np * np).blocks : nt * nt * nt;
}

void launch_gather_kick_drift(uint32_t* xq, int32_t* pq, const uint32_t* id, const float* fmesh,
                              long fStride, const Lattice& L, const Bins& b, float kick,
                              float drift, int do_drift, uint32_t* ck_x, int32_t* ck_p,
                              unsigned* ovf, bool count_bins, hipStream_t s) {
    GatherArgs A{};
    A.ovf = ovf;
    A.count = count_bins && do_drift;
    A.xq = xq;
    A.pq = pq;
    A.id = id;
    A.mesh = fmesh;
    A.mStride = fStride;
    A.pitch = L.rp;
    A.coeff = kick;
    A.drift = drift;
    A.flag = do_drift;
    A.ck_x = ck_x;
    A.ck_p = ck_p;
    gather_dispatch<kKickDrift>(A, L, b, s);
}

void launch_gather_force(const uint32_t* xq, const float* fmesh, long fStride, const Lattice& L,
                         const Bins& b, float* out, hipStream_t s) {
    GatherArgs A{};
    A.xq = const_cast<uint32_t*>(xq);
    A.mesh = fmesh;
    A.mStride = fStride;
    A.pitch = L.rp;
    A.out = out;
    gather_dispatch<kForce>(A, L, b, s);
}

void launch_unkick_vjp(const uint32_t* xq, int32_t* pq, const float* fmesh, long fStride,
                       const Lattice& L, const Bins& b, float coeff, const float* pi, float* xi,
                       bool xi_zero, double* partials, hipStream_t s) {
    GatherArgs A{};
    A.flag = xi_zero ? 1 : 0;
    A.xq = const_cast<uint32_t*>(xq);
    A.pq = pq;
    A.mesh = fmesh;
    A.mStride = fStride;
    A.pitch = L.rp;
    A.coeff = coeff;
    A.pi_in = pi;
    A.xi = xi;
    A.partials = partials;
    gather_dispatch<kUnkickVjp>(A, L, b, s);
}

void launch_wgrad(const float* mesh, long pitch, float g_scale, uint32_t* xq, const int32_t* pq,
                  float* xi, float* pi, const Lattice& L, const Bins& b, float drift, int mode,
                  double* partials, hipStream_t s, bool dense, bool count_bins, float* pmax) {
    GatherArgs A{};
    A.pmax = pmax;
    A.count = count_bins && mode == 1;
    A.xq = xq;
    A.pq = const_cast<int32_t*>(pq);
    A.mesh = mesh;
    A.pitch = pitch;
    A.dense = dense ? 1 : 0;
    A.coeff = g_scale;
    A.drift = drift;
    A.flag = mode;
    A.xi = xi;
    A.pi = pi;
    A.partials = partials;
    gather_dispatch<kWgrad>(A, L, b, s);
}

void launch_to_fixed_count(const float* disp, uint32_t* xq, const Lattice& L, Bins& b,
                           hipStream_t s) {
    const long P = (long)L.np * L.np * L.np;
    launch_bin_zero(b, s);
    hipLaunchKernelGGL(k_to_fixed_count, dim3(grid_for(P)), dim3(kBlock), 0, s, disp, xq, L, b.tile,
                       P, b.counts, b.keys, b.ranks);
}

void launch_undrift(uint32_t* xq, const int32_t* pq, const float* xi, float* pi, const Lattice& L,
                    const Bins& b, float drift, double* partials, float* pmax, int nblocks,
                    hipStream_t s) {
    const long P = (long)L.np * L.np * L.np;
    hipLaunchKernelGGL(k_undrift, dim3(nblocks), dim3(kBlock), 0, s, xq, pq, xi, pi, L, P, drift,
                       b.tile, b.counts, b.keys, b.ranks, partials, pmax);
}

void launch_final_state(const uint32_t* xq, const int32_t* pq, const uint32_t* id,
                        const Lattice& L, uint32_t* xo, int32_t* po, float* disp, float* mom,
                        hipStream_t s) {
    const long P = (long)L.np * L.np * L.np;
    hipLaunchKernelGGL(k_final_state, dim3(grid_for(P)), dim3(kBlock), 0, s, xq, pq, id, L, P, xo,
                       po, disp, mom);
}

void launch_permute_by_id(const float* in, const uint32_t* id, float* out, long P,
                          hipStream_t s) {
    hipLaunchKernelGGL(k_permute_by_id, dim3(grid_for(P)), dim3(kBlock), 0, s, in, id, out, P);
}

void launch_iota(uint32_t* id, long P, hipStream_t s) {
    hipLaunchKernelGGL(k_iota, dim3(grid_for(P)), dim3(kBlock), 0, s, id, P);
}

void launch_reduce(const double* partials, int nblocks, double* sums, int slot, hipStream_t s) {
    ReduceSets one;
    one.add(partials, nblocks, slot);
    launch_reduce_sets(one, sums, s);
}

void launch_reduce_sets(const ReduceSets& r, double* sums, hipStream_t s) {
    hipLaunchKernelGGL(k_reduce, dim3(r.nsets + (r.maxs ? 1 : 0)), dim3(1024), 0, s, r, sums);
}

void launch_collect(const double* sums, int nsum, const unsigned* words, int nwords,
                    const unsigned* last, double* out, hipStream_t s) {
    hipLaunchKernelGGL(k_collect, dim3((std::max(nsum, nwords + 1) + kBlock - 1) / kBlock),
                       dim3(kBlock), 0, s, sums, nsum, words, nwords, last, out);
}

void launch_recon_err(const uint32_t* a, const uint32_t* id, const uint32_t* b, const Lattice& L,
                      double* partials, int nblocks, unsigned* maxbits, hipStream_t s) {
    const long P = (long)L.np * L.np * L.np;
    hipLaunchKernelGGL(k_recon_err, dim3(nblocks), dim3(kBlock), 0, s, a, id, b, L, P, partials,
                       maxbits);
}

void launch_ic_state(const float* smesh, long sStride, long rp, float D0, float G0,
                     const Lattice& L, uint32_t* xq, int32_t* pq, uint32_t* id, hipStream_t s,
                     const float* s2v, float D2, float G2) {
    const long P = (long)L.np * L.np * L.np;
    hipLaunchKernelGGL(k_ic_state<kIcFixed>, dim3(grid_for(P)), dim3(kBlock), 0, s, smesh, sStride,
                       rp, D0, G0, L, P, xq, pq, id, nullptr, nullptr, s2v, D2, G2);
}

void launch_ic_float(const float* smesh, long sStride, long rp, float D0, float G0,
                     const Lattice& L, float* disp, float* mom, hipStream_t s, const float* s2v,
                     float D2, float G2) {
    const long P = (long)L.np * L.np * L.np;
    hipLaunchKernelGGL(k_ic_state<kIcFloat>, dim3(grid_for(P)), dim3(kBlock), 0, s, smesh, sStride,
                       rp, D0, G0, L, P, nullptr, nullptr, nullptr, disp, mom, s2v, D2, G2);
}

void launch_ic_field(const float* smesh, long sStride, long rp, const Lattice& L, float* out,
                     hipStream_t s) {
    const long P = (long)L.np * L.np * L.np;
    hipLaunchKernelGGL(k_ic_state<kIcField>, dim3(grid_for(P)), dim3(kBlock), 0, s, smesh, sStride,
                       rp, 0.f, 0.f, L, P, nullptr, nullptr, nullptr, out, nullptr, nullptr, 0.f,
                       0.f);
}

void launch_ic_adjoint(float* smesh, long sStride, long rp, float D0, float G0, const Lattice& L,
                       const uint32_t* xq, const int32_t* pq, const uint32_t* id, const float* xi,
                       const float* pi, double* partials, int nblocks, unsigned* maxbits,
                       hipStream_t s, const float* s2v, float* s2_bar, float D2, float G2) {
    const long P = (long)L.np * L.np * L.np;
    auto k = s2v ? k_ic_adjoint<true> : k_ic_adjoint<false>;
    hipLaunchKernelGGL(k, dim3(nblocks), dim3(kBlock), 0, s, smesh, sStride, rp, D0, G0, L, P, xq,
                       pq, id, xi, pi, partials, maxbits, s2v, s2_bar, D2, G2);
}

void launch_lpt_pointwise(const float* a, const float* b, const float* c, float* out, int n,
                          long rp, int op, float scale, hipStream_t s) {
    const long N = (long)n * n * n;
    hipLaunchKernelGGL(k_lpt_pointwise, dim3(grid_for(N)), dim3(kBlock), 0, s, a, b, c, out, n,
                       rp, op, scale);
}

void launch_add_from_pitched(const float* src, float* dst, int n, long rp, float scale,
                             hipStream_t s) {
    const long N = (long)n * n * n;
    hipLaunchKernelGGL(k_add_from_pitched, dim3(grid_for(N)), dim3(kBlock), 0, s, src, dst, n, rp,
                       scale);
}

void launch_dot_pitched(const float* src, const float* b, int n, long rp, double* partials,
                        int nblocks, hipStream_t s) {
    hipLaunchKernelGGL(k_dot_pitched, dim3(nblocks), dim3(kBlock), 0, s, src, b, n, rp, partials);
}

void launch_deinterleave(const float* v, float* dst, long dstStride, int np, long rp,
                         hipStream_t s) {
    const long P = (long)np * np * np;
    hipLaunchKernelGGL(k_deinterleave, dim3(grid_for(P)), dim3(kBlock), 0, s, v, dst, dstStride, np,
                       rp);
}

void launch_mse(const float* d, const float* t, float* g, long n3, double* partials,
                int nblocks, hipStream_t s) {
    hipLaunchKernelGGL(k_mse, dim3(nblocks), dim3(kBlock), 0, s, d, t, g, n3, (float)(2.0 / n3),
                       partials);
}

void launch_pk_loss(const double* bins, const double* target, int nbins, double norm, double weight,
                    double* out, float* table, int* finite, hipStream_t s) {
    hipLaunchKernelGGL(k_pk_loss, dim3(1), dim3(kBlock), 0, s, bins, target, nbins, norm, weight,
                       out, table, finite);
}

void launch_mse_periodic(const float* a, const float* b, float* g, long n, float box, float gscale,
                         double* partials, int nblocks, hipStream_t s) {
    hipLaunchKernelGGL(k_mse_periodic, dim3(nblocks), dim3(kBlock), 0, s, a, b, g, n, box,
                       1.f / box, gscale, partials);
}

}  // namespace pmx
