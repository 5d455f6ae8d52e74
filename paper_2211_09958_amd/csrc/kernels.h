// Internal launchers of the libpmx HIP kernels (not part of the public ABI).
//
// Mesh storage: a complex half-spectrum buffer holds [n][n][cs] float2 with
// cs >= n/2 + 1 (a multiple of 16, so every row starts 128-byte aligned).  The
// same buffer viewed as reals holds a real mesh [n][n][rp] with row pitch
// rp = 2 cs floats; the x-axis (last, contiguous) transforms run in place on
// those rows.  Axis 0 is the slowest.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace pmx {

inline int complex_row_stride(int n) { return ((n / 2 + 1) + 15) / 16 * 16; }

// Twiddle tables on the device: w[m] = exp(-2 pi i m / n) (real-split
// post-twiddles of the last-axis passes) and the per-stage tables of
// fft_plan.h (kStageTableSize entries).
struct Twiddles {
    const float2* w;
    int n;
    const float2* stages;
};
// Host: fill the per-stage twiddle table (kStageTableSize entries).
void fill_stage_twiddles(float2* table);
// Compute units of the current device (work-groups of the persistent kernels).
int device_cus();

// ---------------------------------------------------------------- FFT
// Meshes up to kMaxPlane per side take their axis-2 and axis-1 transforms in one
// launch (a plane per work-group); larger ones in a pass per axis.
constexpr int kMaxPlane = 64;
// Axes 2 and 1 of `nbuf` buffers `bufStride` float2 apart, in place: real rows ->
// half spectra transformed along both (r2c), and back (c2r).  With `real` (one
// buffer) the real rows are read from, or written to, a dense [n]^3 array in
// plain row order.  c2r with `real` and `open`: nothing is written to `real` when
// *open, on the device, is 0.
void launch_fft_xy_r2c(const float* real, float2* buf, int n, int cs, int nbuf, long bufStride,
                       const Twiddles& tw, hipStream_t s);
void launch_fft_yx_c2r(float2* buf, float* real, int n, int cs, int nbuf, long bufStride,
                       const Twiddles& tw, hipStream_t s, const int* open = nullptr);
// n <= kMaxPlane: three real buffers -> S_0 in the first and n1 S_1 + k2 S_2 in
// the second (the inputs of launch_grad_adj_z)
void launch_plane_r2c_merge(float2* buf, int n, int cs, long bufStride, const Twiddles& tw,
                            hipStream_t s);
// n <= kMaxPlane: the outputs of launch_grad_z, F~_0 in the first of three buffers
// and G in `g` (a buffer of its own), -> the three real force meshes
void launch_plane_c2r_force(float2* buf, const float2* g, int n, int cs, long bufStride,
                            const Twiddles& tw, hipStream_t s);
// The passes of axis 2 or axis 1 alone take n > kMaxPlane only.
// Real rows -> half spectra along the last axis, in place, for `nbuf` buffers
// `bufStride` float2 apart.  Unnormalised exp(-i k x).
void launch_fft_x_r2c(float2* buf, int n, int cs, int nbuf, long bufStride, const Twiddles& tw, hipStream_t s);
// The same with the real rows read from a dense [n]^3 array in plain row order
// (4-byte aligned) and the half spectra written to `buf`.
void launch_fft_x_r2c_from(const float* real, float2* buf, int n, int cs, const Twiddles& tw,
                           hipStream_t s);
// Inverse of the above without the 1/n factor (Hermitian rows assumed).
void launch_fft_x_c2r(float2* buf, int n, int cs, int nbuf, long bufStride, const Twiddles& tw, hipStream_t s);
// The same with the real rows written to a dense [n]^3 array in plain row order
// (unless `open` is given and *open is 0).
void launch_fft_x_c2r_to(float2* buf, float* real, int n, int cs, const Twiddles& tw,
                         hipStream_t s, const int* open = nullptr);
// as launch_fft_x_c2r, with buffer kmul_buf multiplied by i k2 first
void launch_fft_x_c2r_dk2(float2* buf, int n, int cs, int nbuf, long bufStride, int kmul_buf,
                          const Twiddles& tw, hipStream_t s);
// inverse axis-1 pass of G: out_g = IFFT_1(G), g <- IFFT_1(i n1 G)
void launch_fft_y_split(float2* g, float2* out_g, int n, int cs, const Twiddles& tw,
                        hipStream_t s);
// forward axis-1 pass merging two spectra: g1 <- n1 FFT_1(g1) + k2 FFT_1(g2)
// (n1 the axis-1 frequency, zero on its Nyquist plane; k2 zero on the Nyquist
// column): the input of launch_grad_adj_z's second spectrum
void launch_fft_y_merge(float2* g1, const float2* g2, int n, int cs, const Twiddles& tw,
                        hipStream_t s);
// Complex transform along axis 1, in place; dir = -1 forward, +1 inverse.
void launch_fft_y(float2* buf, int n, int cs, int dir, int nbuf, long bufStride,
                  const Twiddles& tw, hipStream_t s);
// Fused axis-0 pass of the force: forward axis-0 FFT of src (already
// transformed along axes 2 and 1), then dst = IFFT_0(i n0 radial delta) (zero
// on the Nyquist plane of axis 0) and dst_g = G = IFFT_0(radial delta);
// launch_fft_y_split and launch_fft_x_c2r_dk2, or launch_plane_c2r_force, turn G
// into the axis-1 and axis-2 components.
void launch_grad_z(const float2* src, float2* dst, float2* dst_g, int n, int cs,
                   const float* radial, const Twiddles& tw, hipStream_t s);
// Fused axis-0 pass of the transpose: dst = inverse-axis-0 of
// Sum_j conj(M_j) forward-axis-0(G_j), with M_j = i n_j radial, given G_0 at src
// and n1 G_1 + n2 G_2 (from launch_fft_y_merge) at src + srcStride, both
// already transformed along axes 2 and 1.  dst may equal the `dens` buffer.
// When fbar != nullptr also forms
// fbar[|n|^2] = Sum mult * Sum_j Re(conj(G_j) i n_j fscale/|n|^2 dens_k)
// (mult = 1 on the k2 = 0, n/2 planes, else 2) using forward-axis-0(dens), with
// `modes` (a complex buffer's size, overlapping none of the others) for the terms
// and their partial sums.
void launch_grad_adj_z(const float2* src, long srcStride, float2* dst, const float2* dens,
                       int n, int cs, const float* radial, float* fbar, float* modes,
                       float fscale, const Twiddles& tw, hipStream_t s);
// Full 3-D transforms between a dense real mesh [n]^3 and a dense half spectrum
// [n][n][n/2+1], through `buf`; the first and last pass read and write the
// caller's layout.  R2C with spec == nullptr leaves the spectrum in `buf`.
void launch_fft3_r2c_dense(const float* real, float2* buf, float2* spec, int n, int cs,
                           const Twiddles& tw, hipStream_t s);
void launch_fft3_c2r_dense(const float2* spec, float2* buf, float* real, int n, int cs,
                           const Twiddles& tw, hipStream_t s);

// Shell sums of the transform of a dense real mesh: bins[3(b-1) + {0,1,2}] =
// {Sum w |d_k|^2, Sum w |n|, Sum w} for b = round(|n|) in [1, nbins], nbins <= n.
// `part`, of the buffer's size, holds partial sums: a buffer of its own leaves
// the spectrum transformed along axes 2 and 1 in `buf`; it may be `buf` itself.
void launch_fft_shells(const float* real, float2* buf, float2* part, int n, int cs, int nbins,
                       double* bins, const Twiddles& tw, hipStream_t s);
// real = unnormalised inverse DFT of table[b - 1] d_k (0 off the shells) for the
// spectrum that launch_fft_shells left in `buf`; table has nbins values.  Nothing is
// written to `real` when *open is 0.
void launch_fft_shell_scale(float2* buf, float* real, int n, int cs, int nbins, const float* table,
                            const int* open, const Twiddles& tw, hipStream_t s);

// ---------------------------------------------------------------- particles
// Particle state is fixed point so that kick and drift are exactly invertible:
// positions x are uint32 in units of box / 2^32 (periodic wrap is integer
// overflow; a mesh cell is 2^shift units), momenta are int32 in units of
// mom_unit = cell * 2^-22, coarsened by powers of two for small cells so that the
// range 2^31 mom_unit covers |p| <= 100 Mpc/h per unit time (state_units).
struct Lattice {
    int np;            // particles per side
    int ng;            // mesh cells per side
    int ratio;         // ng / np
    float inv_cell;    // ng / box
    long rp;           // real-row pitch of meshes (floats)
    int shift;         // 32 - log2(ng)
    uint32_t half;     // half a cell in position units
    uint32_t qstep;    // lattice spacing in position units (2^32 / np)
    float frac;        // 2^-shift
    float len_to_pos;  // 2^32 / box
    float pos_to_len;  // box / 2^32
    float mom_unit;    // momentum per integer unit
    float inv_mom_unit;
};

struct Bins {
    int tile;        // tile side in cells
    int nt;          // tiles per side
    uint32_t* counts;   // [nt^3 * 8 + 1]
    uint32_t* offsets;  // [nt^3 * 8 + 1]
    uint32_t* keys;     // [P]
    uint32_t* ranks;    // [P]
    uint32_t* ord;      // [P] storage slot of the k-th particle in bin order
    uint32_t* scan_tmp; // scan block sums
    // The counts are zero between calls: zeroed in pm_init, and every sort's counts
    // are cleared by the same call's later kernels.  dirty: they may not be, since a
    // call failed in between or particles were counted that are not sorted
    bool dirty = false;
    long nkeys() const { return (long)nt * nt * nt * 8; }
};

void launch_zero(void* p, size_t bytes, hipStream_t s);
int choose_tile(int ng);
long scan_tmp_elems(long nkeys);

// The per-particle arrays that move together when the particles are re-sorted, from
// src to dst: positions, momenta and ids (3, 3 and 1 words per particle), and with
// `cotangents` also xi and pi (3 words each).
struct Records {
    const uint32_t* src[5] = {};
    uint32_t* dst[5] = {};
    bool cotangents = false;
    // with cotangents, sources in lattice order: the ids are the slots and are not
    // read, and a null xi or pi stands for zeros (pi: not written either when its
    // destination is null)
    bool lattice = false;
    void set(int k, const void* from, void* to) {
        src[k] = static_cast<const uint32_t*>(from);
        dst[k] = static_cast<uint32_t*>(to);
    }
    void state(const uint32_t* x, uint32_t* x_to, const int32_t* p, int32_t* p_to,
               const uint32_t* id, uint32_t* id_to) {
        set(0, x, x_to);
        set(1, p, p_to);
        set(2, id, id_to);
    }
    void add_cotangents(const float* xi, float* xi_to, const float* pi, float* pi_to,
                        bool from_lattice) {
        set(3, xi, xi_to);
        set(4, pi, pi_to);
        cotangents = true;
        lattice = from_lattice;
    }
};

// Counting sort of particles by (tile of the CIC base cell, spill class): bin
// offsets and the sorted order b.ord (bin k of the offsets holds the particles
// in storage slots ord[offsets[k]], ..., ord[offsets[k + 1] - 1]); the records
// stay where they are.
// kCounted: the counts, keys and ranks were already produced by the gather that
// moved the particles (see count_bins below) and only the scan and the order
// remain; kCountedOnce: by launch_to_fixed_count, in the order of its waves.
enum Counted { kNotCounted, kCounted, kCountedOnce };
void launch_bin(const uint32_t* xq, const Lattice& L, Bins& b, Counted counted, hipStream_t s);
// Zeroes the bin counts ahead of a kernel that counts particles, if they are dirty.
inline void launch_bin_zero(Bins& b, hipStream_t s) {
    if (!b.dirty) return;
    launch_zero(b.counts, (b.nkeys() + 1) * sizeof(uint32_t), s);
    // a capture only records the clearing, and may never be replayed
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) == hipSuccess && st == hipStreamCaptureStatusNone)
        b.dirty = false;
}
// Moves every record array from src to dst in the order b.ord and resets b.ord
// to the identity (each bin then a contiguous range of the records).
void launch_compact(Bins& b, const Records& rec, long P, hipStream_t s);
// Density delta = rho - 1 (particle mass (ng/np)^3) into a real mesh with pitch
// L.rp (nullable) and/or a caller's dense [ng]^3 array in plain order (nullable,
// any 4-byte alignment); every cell written once (no pre-zeroing), deterministic.
// Follows a launch_bin (whose counts it clears where that has not).
void launch_scatter_density(const uint32_t* xq, const Lattice& L, const Bins& b, float* mesh,
                            float* dense, hipStream_t s);
// out_j = Sum_p coeff v_{p,j} w(x_p, node) for j = 0..2 into meshes out + j*outStride
// (64-bit fixed point, bitwise reproducible); *vmax holds max |v| as float bits
// (launch_absmax, or the maxima of the kernel that wrote v).
void launch_scatter_vec(const uint32_t* xq, const float* v, float coeff, const unsigned* vmax,
                        const Lattice& L, const Bins& b, float* out, long outStride,
                        hipStream_t s);

// *out = max(*out, max |v| over n floats), as float bits.
void launch_absmax(const float* v, long n, unsigned* out, hipStream_t s);

// Gathers: one work-group per tile of the current bins, or for few particles per
// cell a grid over the storage slots (the particles' state is read and written in
// their storage slots); partials (nullable) get one FP64 value per work-group,
// gather_partials(np, ng) values.
long gather_partials(int np, int ng);
// F = gather(force meshes), p += kick F, optional checkpoint copy of (x, p) in
// lattice order (by id), then x += drift p (if do_drift).  *ovf (nullable) is
// set to 1 when a new momentum does not fit the int32 fixed-point range.
// With count_bins (and do_drift), the drifted particles are also counted into
// b's counts, keys and ranks for the next launch_bin(kCounted), after a
// launch_bin_zero.
void launch_gather_kick_drift(uint32_t* xq, int32_t* pq, const uint32_t* id, const float* fmesh,
                              long fStride, const Lattice& L, const Bins& b, float kick,
                              float drift, int do_drift, uint32_t* ck_x, int32_t* ck_p,
                              unsigned* ovf, bool count_bins, hipStream_t s);
// out[p][j] = Sum w F_j for the particle in storage slot p.
void launch_gather_force(const uint32_t* xq, const float* fmesh, long fStride, const Lattice& L,
                         const Bins& b, float* out, hipStream_t s);
// Reverse step at x: F = gather; p -= coeff F (exact inverse of the forward
// kick; pq nullable); xi (taken as zero with xi_zero) += coeff Sum_j pi_j grad w .
// F~_j; partials Sum pi . F.  pi null: zero, xi is then neither read nor written.
void launch_unkick_vjp(const uint32_t* xq, int32_t* pq, const float* fmesh, long fStride,
                       const Lattice& L, const Bins& b, float coeff, const float* pi, float* xi,
                       bool xi_zero, double* partials, hipStream_t s);
// xi += g_scale Sum grad w . mesh (mesh row pitch given; rows in the workspace
// order of layout.h, or in plain order when dense).  mode 1 also does the rest
// of a reverse step: partials Sum xi . p, pi += drift xi, x -= drift p (exact
// inverse of the forward drift); mode 2 only updates xi.
// count_bins (mode 1): the un-drifted particles are counted as in
// launch_gather_kick_drift.  pmax (mode 1, nullable): max |pi| of the new pi, one
// value per partial.
void launch_wgrad(const float* mesh, long pitch, float g_scale, uint32_t* xq, const int32_t* pq,
                  float* xi, float* pi, const Lattice& L, const Bins& b, float drift, int mode,
                  double* partials, hipStream_t s, bool dense = false, bool count_bins = false,
                  float* pmax = nullptr);
// The rest of a reverse step where pi was zero and the force transpose adds
// nothing to xi: pi = drift xi, x -= drift p, block partials of Sum xi . p, the
// un-drifted particles counted into b and max |pi| per block in pmax (as
// launch_wgrad with count_bins and pmax).
void launch_undrift(uint32_t* xq, const int32_t* pq, const float* xi, float* pi, const Lattice& L,
                    const Bins& b, float drift, double* partials, float* pmax, int nblocks,
                    hipStream_t s);
// Displacements (float, Mpc/h, lattice order) -> fixed-point positions q + s in
// lattice order, counted into b's counts, keys and ranks for a following
// launch_bin(kCountedOnce).
void launch_to_fixed_count(const float* disp, uint32_t* xq, const Lattice& L, Bins& b,
                           hipStream_t s);
// Fixed-point state (any order) -> lattice order: displacement (minimum image of
// x - q) and momentum, and the fixed-point state itself.
void launch_final_state(const uint32_t* xq, const int32_t* pq, const uint32_t* id,
                        const Lattice& L, uint32_t* xo, int32_t* po, float* disp, float* mom,
                        hipStream_t s);
// [P][3] float records to lattice order: out[id[k]] = in[k].
void launch_permute_by_id(const float* in, const uint32_t* id, float* out, long P,
                          hipStream_t s);
void launch_iota(uint32_t* id, long P, hipStream_t s);
int particle_blocks(long P);

// sums[slot] = Sum of partials[0..nblocks)
void launch_reduce(const double* partials, int nblocks, double* sums, int slot, hipStream_t s);
// The same for several sets of partials in one launch, and with maxs also *vmax =
// max of nmax non-negative floats, as float bits.
struct ReduceSets {
    int nsets = 0;
    const double* src[9];
    int n[9], slot[9];
    const float* maxs = nullptr;
    int nmax = 0;
    unsigned* vmax = nullptr;
    void add(const double* partials, int count, int to) {
        src[nsets] = partials;
        n[nsets] = count;
        slot[nsets++] = to;
    }
};
void launch_reduce_sets(const ReduceSets& r, double* sums, hipStream_t s);
// out[0..nsum) = sums, then as 32-bit words words[0..nwords) and *last; out is host
// memory mapped to the device.
void launch_collect(const double* sums, int nsum, const unsigned* words, int nwords,
                    const unsigned* last, double* out, hipStream_t s);
// Reconstruction error of fixed-point positions in cells: partials of
// Sum_k |a[k] - b[id[k]]|^2 (minimum image), *maxbits (as float bits) = max.
void launch_recon_err(const uint32_t* a, const uint32_t* id, const uint32_t* b, const Lattice& L,
                      double* partials, int nblocks, unsigned* maxbits, hipStream_t s);

// Zel'dovich state from three real meshes s_j (pitch rp, on the particle
// lattice): x = q + D0 s, p = G0 s in fixed point; with s2v ([P][3] lattice order,
// 2LPT) the state adds D2 s2 and G2 s2.  launch_ic_float writes the same state
// as displacement x - q and momentum, launch_ic_field s itself ([P][3]).
void launch_ic_state(const float* smesh, long sStride, long rp, float D0, float G0,
                     const Lattice& L, uint32_t* xq, int32_t* pq, uint32_t* id, hipStream_t s,
                     const float* s2v = nullptr, float D2 = 0.f, float G2 = 0.f);
void launch_ic_float(const float* smesh, long sStride, long rp, float D0, float G0,
                     const Lattice& L, float* disp, float* mom, hipStream_t s,
                     const float* s2v = nullptr, float D2 = 0.f, float G2 = 0.f);
void launch_ic_field(const float* smesh, long sStride, long rp, const Lattice& L, float* out,
                     hipStream_t s);
// The state and cotangents at x_0 (sorted order) against the ICs: block partials,
// set k at k nblocks, of
//   0 Sum|dx|^2 (cells^2)  1 Sum|dp|^2  2 Sum|p|^2 (fixed-point units)
//   3 Sum xi.s  4 Sum pi.s  5 Sum s_bar.s, s_bar = D0 xi + G0 pi
//   6 Sum xi.s2  7 Sum pi.s2  8 Sum s2_bar.s2, s2_bar = D2 xi + G2 pi (2LPT, s2v given)
// and max |dx| (cells) into *maxbits.  s_bar replaces s in the meshes, s2_bar goes
// to [P][3] in lattice order.
void launch_ic_adjoint(float* smesh, long sStride, long rp, float D0, float G0, const Lattice& L,
                       const uint32_t* xq, const int32_t* pq, const uint32_t* id, const float* xi,
                       const float* pi, double* partials, int nblocks, unsigned* maxbits,
                       hipStream_t s, const float* s2v = nullptr, float* s2_bar = nullptr,
                       float D2 = 0.f, float G2 = 0.f);
// Axis-0 pass with a 2LPT multiplier w of integer wave numbers nv, m2 = |n|^2, R =
// table[m2] (or 1/m2 when table is null): mode 0 nv[a] nv[b] R (0 on the Nyquist
// plane of a or b when a != b), mode 1 (m2 - nv[a]^2) R, mode 2 m2 table[m2]; times
// scale, 0 at m2 = 0.  dir = +1: dst = inverse transform of w src; dir = -1: dst =
// w times the forward transform of src, or += when accumulate (dst and src
// distinct).
void launch_fft_z_mul(const float2* src, float2* dst, int n, int cs, int dir, int ax_a, int ax_b,
                      int mode, const float* table, float scale, bool accumulate,
                      const Twiddles& tw, hipStream_t s);
// Real meshes of one layout: op 0 out = ab + ac + bc; op 1 out = a - b^2 (- c^2
// if c); op 2 out = scale a b.  out may alias a.
void launch_lpt_pointwise(const float* a, const float* b, const float* c, float* out, int n,
                          long rp, int op, float scale, hipStream_t s);
// dst [n]^3 += scale * pitched src; block partials of Sum pitched src * b.
void launch_add_from_pitched(const float* src, float* dst, int n, long rp, float scale,
                             hipStream_t s);
void launch_dot_pitched(const float* src, const float* b, int n, long rp, double* partials,
                        int nblocks, hipStream_t s);
// AoS [P][3] component j -> pitched mesh j (three meshes).
void launch_deinterleave(const float* v, float* dst, long dstStride, int np, long rp,
                         hipStream_t s);
// Loss L = n^-3 Sum (d - t)^2 partials, g = 2 (d - t) / n^3 (nullable).
void launch_mse(const float* d, const float* t, float* g, long n3, double* partials,
                int nblocks, hipStream_t s);
// P(k) loss from launch_fft_shells' bins: with P_b = norm bins[3b]/bins[3b+2] and
// the shells that hold modes and a nonzero finite target,
// out[0] = weight mean_b (P_b / target_b - 1)^2, out[1] = the sum of the squares,
// *finite = whether that is finite, and table[b] = 2 norm / bins[3b+2] dL/dP_b (0 on
// the other shells).
void launch_pk_loss(const double* bins, const double* target, int nbins, double norm, double weight,
                    double* out, float* table, int* finite, hipStream_t s);
// block partials of Sum (minimum-image a - b)^2; g = gscale * (a - b) wrapped (nullable)
void launch_mse_periodic(const float* a, const float* b, float* g, long n, float box, float gscale,
                         double* partials, int nblocks, hipStream_t s);

// Filter network (2-64-64-1 SiLU) at sf.n scale factors, table t at offset t stride:
// radial[n2] = (1 + g(|k|/kNyq, a)) * base(n2) with base(n2) = fscale / n2 (0 at
// n2 = 0); also table = 1 + g (both nullable).
constexpr int kMaxTables = 32;
struct ScaleFactors {
    int n = 0;
    float a[kMaxTables];
    void add(double v) { a[n++] = (float)v; }
};
void launch_mlp_table(const float* theta, int n, const ScaleFactors& sf, float fscale, long stride,
                      float* radial, float* table, hipStream_t s);
// dL/dtheta += backprop of the sf.n tables fbar[n2] (dL/df) through the network.
void launch_mlp_backward(const float* theta, int n, const ScaleFactors& sf, long stride,
                         const float* fbar, float* gtheta, float* scratch, hipStream_t s);
long mlp_backward_scratch(int n);
// Adam step on the mean of ngrad gradients g[ngrad][n]
void launch_adam(float* p, const float* g, int ngrad, float* m, float* v, int n, float lr,
                 float b1, float b2, float eps, float bc1, float bc2, hipStream_t s);

// Message returned by pm_last_error(NULL) (calls without a context).
void set_context_free_error(const char* msg);

}  // namespace pmx
