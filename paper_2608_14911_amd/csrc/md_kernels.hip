// gfx950 kernels of the per-timestep short-range MD step (ESPResSo++,
// arXiv 2608.14911): cell binning and stable cell sort (CellGrid, section
// "Software design"), Verlet-list build with a skin (VerletList +
// system.skin, section "Example usage"), LJ / capped-LJ pair forces
// (LennardJones, LennardJonesCapped with shift='auto'), FENE + cosine
// bending bonded forces (bonded interactions, section "Functionality"),
// velocity Verlet with the Langevin force (VelocityVerlet +
// LangevinThermostat) and FP64 energy / virial reductions
// (computeEnergy()).
//
// Layout: particles are kept sorted by cell so that a wavefront's 64 lanes
// stream neighbouring particles; positions are double4 (x, y, z, type) and
// fixed-point int4 (qx, qy, qz, type), so a gathered neighbour is one 32- or
// 16-byte segment; velocities and build positions are SoA planes; the
// Verlet list is ELL in tiles of 64 particles (entry k of particle i at
// (i / 64) * cap * 64 + k * 64 + i % 64), so that the 64 lanes of a
// wavefront read 256 contiguous bytes per entry.
#include "md_device.h"


namespace md {

// ------------------------------------------------------------------ helpers

// Minimum image d - L rint(d / L), branch-free.  For |d| < L (positions in
// [0, L)) the shift is 0 or +-L and the result is d -/+ L rounded once, the
// same value a compare-and-shift gives except within an ulp of |d| = L/2,
// which is never inside the list radius (L >= 3 cells >= 2 rv).  Exactly
// antisymmetric: d_ji = -d_ij.
__device__ __forceinline__ double mimg(double d, double L, double invL) {
    return fma(-L, rint(d * invL), d);
}

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

__device__ __forceinline__ void cell_coords(const Geom& g, double x, double y, double z, int& cx,
                                            int& cy, int& cz) {
    // positions are in [0, L); the clamp covers rounding at L and NaN
    double fx = x * g.invh[0], fy = y * g.invh[1], fz = z * g.invh[2];
    cx = (fx >= 0.0) ? (int)fx : 0;
    cy = (fy >= 0.0) ? (int)fy : 0;
    cz = (fz >= 0.0) ? (int)fz : 0;
    cx = clampi(cx, 0, g.nc[0] - 1);
    cy = clampi(cy, 0, g.nc[1] - 1);
    cz = clampi(cz, 0, g.nc[2] - 1);
}

__device__ __forceinline__ uint32_t cell_of(const Geom& g, const double4& p) {
    int cx, cy, cz;
    cell_coords(g, p.x, p.y, p.z, cx, cy, cz);
    return (uint32_t)(((int64_t)cz * g.nc[1] + cy) * g.nc[0] + cx);
}

// Philox4x64-10 (Salmon, Moraes, Dror, Shaw, SC'11): 10 rounds of two
// 64x64->128 multiplies with the published multipliers, key bumped by the
// published Weyl constants between rounds.
__device__ __forceinline__ void philox4x64_10(uint64_t& x0, uint64_t& x1, uint64_t& x2, uint64_t& x3,
                                              uint64_t k0, uint64_t k1) {
    const uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        uint64_t hi0 = __umul64hi(M0, x0), lo0 = M0 * x0;
        uint64_t hi1 = __umul64hi(M1, x2), lo1 = M1 * x2;
        uint64_t n0 = hi1 ^ x1 ^ k0;
        uint64_t n2 = hi0 ^ x3 ^ k1;
        x0 = n0;
        x1 = lo1;
        x2 = n2;
        x3 = lo0;
        k0 += 0x9E3779B97F4A7C15ull;
        k1 += 0xBB67AE8584CAA73Bull;
    }
}

// Philox4x32-10 (the same paper): four 32-bit words, 10 rounds of two
// 32x32->64 multiplies with the published multipliers, the key bumped by the
// published Weyl constants between rounds.
__device__ __forceinline__ void philox4x32_10(uint32_t& x0, uint32_t& x1, uint32_t& x2, uint32_t& x3,
                                              uint32_t k0, uint32_t k1) {
    const uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint32_t hi0 = __umulhi(M0, x0), lo0 = M0 * x0;
        const uint32_t hi1 = __umulhi(M1, x2), lo1 = M1 * x2;
        const uint32_t n0 = hi1 ^ x1 ^ k0;
        const uint32_t n2 = hi0 ^ x3 ^ k1;
        x0 = n0;
        x1 = lo1;
        x2 = n2;
        x3 = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
}

// Three N(0,1) draws keyed (seed, stream) at counter (step, tag, 0, 0):
// uniforms ((w >> 11) + 1/2) 2^-53 in (0,1), Box-Muller in FP64.
__device__ __forceinline__ void gauss3(uint64_t seed, uint64_t stream, uint64_t step, uint64_t tag,
                                       double& g0, double& g1, double& g2) {
    uint64_t x0 = step, x1 = tag, x2 = 0, x3 = 0;
    philox4x64_10(x0, x1, x2, x3, seed, stream);
    const double two_pi = 6.283185307179586;
    double u0 = ((double)(x0 >> 11) + 0.5) * 0x1.0p-53;
    double u1 = ((double)(x1 >> 11) + 0.5) * 0x1.0p-53;
    double u2 = ((double)(x2 >> 11) + 0.5) * 0x1.0p-53;
    double u3 = ((double)(x3 >> 11) + 0.5) * 0x1.0p-53;
    double r0 = sqrt(-2.0 * log(u0));
    double r1 = sqrt(-2.0 * log(u2));
    g0 = r0 * cos(two_pi * u1);
    g1 = r0 * sin(two_pi * u1);
    g2 = r1 * cos(two_pi * u3);
}

template <typename Real>
__device__ __forceinline__ Real rcp(Real x);
template <>
__device__ __forceinline__ float rcp<float>(float x) { return __builtin_amdgcn_rcpf(x); }
template <>
__device__ __forceinline__ double rcp<double>(double x) { return 1.0 / x; }

template <typename Real>
__device__ __forceinline__ Real rsq(Real x);
template <>
__device__ __forceinline__ float rsq<float>(float x) { return __builtin_amdgcn_rsqf(x); }
template <>
__device__ __forceinline__ double rsq<double>(double x) { return 1.0 / sqrt(x); }

template <typename Real>
__device__ __forceinline__ Real logr(Real x);
template <>
__device__ __forceinline__ float logr<float>(float x) { return logf(x); }
template <>
__device__ __forceinline__ double logr<double>(double x) { return log(x); }

template <typename Real>
__device__ __forceinline__ const PairCoef<Real>& coef(const PairTable& pt, int tp);
template <>
__device__ __forceinline__ const PairCoef<float>& coef<float>(const PairTable& pt, int tp) { return pt.f[tp]; }
template <>
__device__ __forceinline__ const PairCoef<double>& coef<double>(const PairTable& pt, int tp) { return pt.d[tp]; }

__device__ __forceinline__ bool rebuild_requested(const Bufs& b, int parity) {
    return __atomic_load_n(&b.ctl->rebuild[parity], __ATOMIC_RELAXED) != 0;
}

// Start of a step, by one thread of the rebuild stage's first kernel: the step
// that ran before it (if its call has not been finalized) ends here; its
// record is left to the step kernel's first block (finalize_body, MODE_PREV),
// where it costs no launch of its own.  The other parity's flag, last read by
// the step before, is cleared for this step's kernel to set.
__device__ __forceinline__ void advance_step(const Bufs& b, int parity) {
    DevCtl* c = b.ctl;
    const int ran = c->ran;
    c->fin_prev = ran;
    if (ran) {
        c->prev_status = c->status;
        c->prev_nl_max = c->nl_max;
        c->prev_rebuilds = c->n_rebuilds;
        c->step += 1;
        c->vel_half = 1;
    }
    c->ran = 1;
    c->rebuild[parity ^ 1] = 0;
}

// ------------------------------------------------------------------ init / state I/O

// Load tag-ordered FP64 state into the (identity-ordered) sorted arrays,
// folding positions into [0, L) with image counters.
__global__ void __launch_bounds__(kBlock) k_init_load(Geom g, Bufs b, int parity, const double* pos,
                                                      const double* vel, const int32_t* type,
                                                      const int32_t* image) {
    const int64_t n = g.n;
    for (int64_t i = gtid(); i < n; i += gstride()) {
        double p[3];
        for (int d = 0; d < 3; ++d) {
            double x = pos[3 * i + d];
            int im = image ? image[3 * i + d] : 0;
            double k = floor(x / g.L[d]);
            if (k != 0.0 && isfinite(k)) {
                x -= k * g.L[d];
                im += (int)k;
            }
            if (x < 0.0) { x += g.L[d]; im -= 1; }
            if (x >= g.L[d]) { x -= g.L[d]; im += 1; }
            p[d] = x;
            b.img[d * n + i] = im;
            b.v[d * n + i] = vel ? vel[3 * i + d] : 0.0;
        }
        int ty = type ? type[i] : 0;
        if (ty < 0 || ty >= g.ntypes) {
            atomicOr(&b.ctl->status, MD_FLAG_BAD_TYPE);
            ty = 0;
        }
        b.x[parity][i] = make_double4(p[0], p[1], p[2], (double)ty);
        b.tag[i] = (int32_t)i;
        b.inv[i] = (int32_t)i;
    }
}

// After a rebuild from the build positions, put the current state into the
// slots the sort assigned (used by md_set_state with a build snapshot).
__global__ void __launch_bounds__(kBlock) k_overwrite_state(Geom g, Bufs b, int parity,
                                                            const double* pos, const double* vel,
                                                            const int32_t* image) {
    const int64_t n = g.n;
    for (int64_t s = gtid(); s < n; s += gstride()) {
        int64_t t = b.tag[s];
        double4 old = b.x[parity][s];
        double p[3];
        for (int d = 0; d < 3; ++d) {
            double x = pos[3 * t + d];
            int im = image ? image[3 * t + d] : 0;
            if (x < 0.0) { x += g.L[d]; im -= 1; }
            if (x >= g.L[d]) { x -= g.L[d]; im += 1; }
            p[d] = x;
            b.img[d * n + s] = im;
            b.v[d * n + s] = vel[3 * t + d];
        }
        b.x[parity][s] = make_double4(p[0], p[1], p[2], old.w);
        const int4 q = quantize4(g, p[0], p[1], p[2], old.w);
        b.xq[parity][s] = q;
        if (g.x3_on) store_q3(b.x3[parity], s, q);
    }
}

__global__ void __launch_bounds__(kBlock) k_get_state(Geom g, Bufs b, int parity, double* pos,
                                                      double* vel, int32_t* image, double* pos_build) {
    const int64_t n = g.n;
    for (int64_t s = gtid(); s < n; s += gstride()) {
        int64_t t = b.tag[s];
        double4 p = b.x[parity][s];
        if (pos) { pos[3 * t] = p.x; pos[3 * t + 1] = p.y; pos[3 * t + 2] = p.z; }
        for (int d = 0; d < 3; ++d) {
            if (vel) vel[3 * t + d] = b.v[d * n + s];
            if (image) image[3 * t + d] = b.img[d * n + s];
            if (pos_build) pos_build[3 * t + d] = b.xb[d * n + s];
        }
    }
}

__global__ void __launch_bounds__(kBlock) k_get_neighbors(Geom g, Bufs b, int32_t* count,
                                                          int32_t* idx, int32_t cap) {
    const int64_t n = g.n;
    for (int64_t s = gtid(); s < n; s += gstride()) {
        int64_t t = b.tag[s];
        int c = b.ncount[s];
        int cc = c < g.cap ? c : g.cap;
        count[t] = c;
        const int32_t* row = b.nl + nl_base(s, g.cap);
        for (int k = 0; k < cc && k < cap; ++k) idx[t * (int64_t)cap + k] = b.tag[row[nl_off(k)]];
    }
}

__global__ void k_set_ctl(Bufs b, int64_t step, int vel_half, int rebuild, int clear_status) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        DevCtl* c = b.ctl;
        if (step >= 0) c->step = step;
        if (vel_half >= 0) c->vel_half = vel_half;
        if (rebuild >= 0) c->rebuild[0] = c->rebuild[1] = (uint32_t)rebuild;
        c->ran = c->fin_prev = 0;
        if (clear_status) { c->status = 0; c->nl_max = 0; }
    }
}

__global__ void __launch_bounds__(kBlock) k_zero_i32(int32_t* p, int64_t n) {
    for (int64_t i = gtid(); i < n; i += gstride()) p[i] = 0;
}

__global__ void __launch_bounds__(kBlock) k_copy_i32(int32_t* dst, const int32_t* src, int64_t n) {
    for (int64_t i = gtid(); i < n; i += gstride()) dst[i] = src[i];
}

// ------------------------------------------------------------------ rebuild: cell sort
// Every rebuild kernel returns at once unless the device flag asks for a
// rebuild, so the whole step can be enqueued (and graph-captured) without a
// host round trip.

// Runs of equal cells over the lanes of a wavefront.  Particles arrive in
// the previous build's cell order, so a run is usually a whole cell's share
// of the wavefront and one atomic serves it.  Active lanes are a prefix of
// the wavefront.  Returns the run's first lane and its length.
__device__ __forceinline__ void cell_run(uint32_t c, bool active, int& first, int& len) {
    const int lane = threadIdx.x & 63;
    const uint32_t prev = __shfl_up(c, 1, 64);
    const uint64_t heads = __ballot(active && (lane == 0 || c != prev));
    // bits 0 .. k: (2 << k) - 1, which is all ones for k = 63
    const uint64_t upto = heads & ((2ull << lane) - 1);
    first = upto ? 63 - __clzll(upto) : 0;
    const uint64_t after = heads & ~((2ull << first) - 1);
    const int nact = __popcll(__ballot(active));
    const int next = after ? __ffsll((unsigned long long)after) - 1 : nact;
    len = next - first;
}

__device__ __forceinline__ uint32_t bin_one(const Geom& g, const Bufs& b, int64_t i, bool active, int parity) {
    uint32_t c = 0xffffffffu;
    if (active) {
        c = cell_of(g, b.x[parity][i]);
        b.cellid[i] = c;
    }
    int first, len;
    cell_run(c, active, first, len);
    if (active && (threadIdx.x & 63) == first) atomicAdd(&b.ccount[c], len);
    return c;
}

// Cells are scanned in kScanBlocks chunks of consecutive cells.  Binning also
// sums each chunk's particles (one atomic per run of equal chunks in a
// wavefront, each chunk's sum on a 128-byte line of its own), so the scan
// needs no separate reduction pass.
__device__ __forceinline__ int64_t scan_chunk_cells(const Geom& g) {
    return (g.ncell + kScanBlocks - 1) / kScanBlocks;
}

__global__ void __launch_bounds__(kBlock) k_bin(Geom g, Bufs b, int parity, int advance) {
    if (advance && gtid() == 0) advance_step(b, parity);
    if (!rebuild_requested(b, parity)) return;
    const int64_t chunk = scan_chunk_cells(g);
    for (int64_t i0 = (int64_t)blockIdx.x * blockDim.x; i0 < g.n; i0 += gstride()) {
        const int64_t i = i0 + threadIdx.x;
        const bool active = i < g.n;
        const uint32_t c = bin_one(g, b, i, active, parity);
        const uint32_t ch = active ? (uint32_t)(c / chunk) : 0xffffffffu;
        int first, len;
        cell_run(ch, active, first, len);
        if (active && (threadIdx.x & 63) == first) atomicAdd(&b.bsum[(int64_t)ch * kChunkPad], len);
    }
}

__device__ int block_exclusive_scan(int v, int& total) {
    __shared__ int wsum[kBlock / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        int y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) wsum[w] = x;
    __syncthreads();
    int off = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < kBlock / 64; ++k) {
        if (k < w) off += wsum[k];
        tot += wsum[k];
    }
    __syncthreads();
    total = tot;
    return off + x - v;
}

__device__ __forceinline__ void scan_chunk(const Geom& g, int blk, int64_t& lo, int64_t& hi) {
    const int64_t chunk = scan_chunk_cells(g);
    lo = blk * chunk;
    hi = lo + chunk;
    if (hi > g.ncell) hi = g.ncell;
    if (lo > g.ncell) lo = g.ncell;
}

__global__ void __launch_bounds__(kBlock) k_scan_reduce(Geom g, Bufs b) {
    if (!rebuild_requested(b, 0)) return;
    int64_t lo, hi;
    scan_chunk(g, blockIdx.x, lo, hi);
    int s = 0;
    for (int64_t c = lo + threadIdx.x; c < hi; c += kBlock) s += b.ccount[c];
    __shared__ int red[kBlock];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = kBlock / 2; o > 0; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) b.bsum[blockIdx.x] = red[0];
}

// Exclusive scan of the kScanBlocks chunk sums by one block.
__global__ void __launch_bounds__(kScanBlocks) k_scan_top(Bufs b) {
    if (!rebuild_requested(b, 0)) return;
    __shared__ int wsum[kScanBlocks / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int v = b.bsum[threadIdx.x];
    int x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) wsum[w] = x;
    __syncthreads();
    int off = 0;
    for (int k = 0; k < w; ++k) off += wsum[k];
    b.bsum[threadIdx.x] = off + x - v;
}

__device__ __forceinline__ void scan_apply_body(const Geom& g, const Bufs& b, int running) {
    int64_t lo, hi;
    scan_chunk(g, blockIdx.x, lo, hi);
    // four consecutive cells per thread and step
    for (int64_t base = lo; base < hi; base += 4 * kBlock) {
        const int64_t c0 = base + 4 * (int64_t)threadIdx.x;
        int v[4], sum = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            v[u] = (c0 + u < hi) ? b.ccount[c0 + u] : 0;
            sum += v[u];
        }
        int tot;
        int e = block_exclusive_scan(sum, tot);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (c0 + u < hi) b.cstart[c0 + u] = running + e;
            e += v[u];
        }
        running += tot;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) b.cstart[g.ncell] = (int32_t)g.n;
}

// Batches: chunk offsets from k_scan_reduce and k_scan_top.
__global__ void __launch_bounds__(kBlock) k_scan_apply(Geom g, Bufs b) {
    if (!rebuild_requested(b, 0)) return;
    scan_apply_body(g, b, b.bsum[blockIdx.x]);
}

// One system: the chunk sums come from k_bin, and each block adds up the
// sums of the chunks before its own (at most kScanBlocks values, read from
// the L2), which replaces the reduction and top-level scan kernels.
__global__ void __launch_bounds__(kBlock) k_scan_chunks(Geom g, Bufs b, int parity) {
    if (!rebuild_requested(b, parity)) return;
    int part = 0;
    for (int k = threadIdx.x; k < (int)blockIdx.x; k += kBlock) part += b.bsum[k * kChunkPad];
    int off;
    (void)block_exclusive_scan(part, off);
    scan_apply_body(g, b, off);
}

// A particle's state into the sort's temporaries at a slot of its cell's segment.
__device__ __forceinline__ void stash(const Bufs& b, int64_t n, int64_t slot, const double4& p, const double (&vv)[3],
                                      const int32_t (&im)[3], int32_t t) {
    b.xt[slot] = p;
    for (int d = 0; d < 3; ++d) {
        b.vt[d * n + slot] = vv[d];
        b.imgt[d * n + slot] = im[d];
    }
    b.tsc[slot] = t;
}

// Scatter into cell segments, one atomic per run of equal cells; counts
// return to zero for the next build.  The whole state moves with its slot, so
// that the pass that orders the cells reads nothing but the temporaries and
// writes the sorted arrays at once.  A pass each for slots, order and the copy
// back took, in the 1,048,576-particle fluid, 23 us per step on average (three
// rebuilds in 20 steps, launches that return included); these two take 17.
__device__ __forceinline__ void scatter_one(const Geom& g, const Bufs& b, int64_t i, bool active, int parity) {
    const int64_t n = g.n;
    const int64_t ii = active ? i : 0;
    const uint32_t c = active ? b.cellid[ii] : 0xffffffffu;
    const double4 p = b.x[parity][ii];
    double vv[3];
    int32_t im[3];
    for (int d = 0; d < 3; ++d) {
        vv[d] = b.v[d * n + ii];
        im[d] = b.img[d * n + ii];
    }
    const int32_t t = b.tag[ii];
    int first, len;
    cell_run(c, active, first, len);
    const int lane = threadIdx.x & 63;
    int top = 0;
    if (active && lane == first) top = atomicSub(&b.ccount[c], len);
    top = __shfl(top, first, 64);
    // the run owns slots [start + top - len, start + top)
    if (active) stash(b, n, b.cstart[c] + top - len + (lane - first), p, vv, im, t);
}

__global__ void __launch_bounds__(kBlock) k_scatter(Geom g, Bufs b, int parity) {
    if (!rebuild_requested(b, parity)) return;
    // the chunk sums were read by the scan: clear them for the next build
    for (int64_t k = gtid(); k < kScanBlocks; k += gstride()) b.bsum[k * kChunkPad] = 0;
    for (int64_t i0 = (int64_t)blockIdx.x * blockDim.x; i0 < g.n; i0 += gstride()) {
        const int64_t i = i0 + threadIdx.x;
        scatter_one(g, b, i, i < g.n, parity);
    }
}

// Order inside a cell by particle tag: the sorted order is then a function
// of the positions alone, so a run resumed from a saved build snapshot
// reproduces it exactly.  From the temporaries to the sorted arrays.
__device__ __forceinline__ void rank_one(const Geom& g, const Bufs& b, int64_t s, int parity, int bonded) {
    const int64_t n = g.n;
    if (s == 0) {
        b.ctl->n_rebuilds += 1;
        b.ctl->nl_max = 0;
        b.ctl->build_step = b.ctl->step;
    }
    // every load before the first store: a load after a store it may
    // alias cannot be moved above it, and would wait in turn
    const double4 p = b.xt[s];
    const int32_t t = b.tsc[s];
    double vv[3];
    int32_t im[3];
    for (int d = 0; d < 3; ++d) {
        vv[d] = b.vt[d * n + s];
        im[d] = b.imgt[d * n + s];
    }
    const uint32_t c = cell_of(g, p);
    const int st = b.cstart[c], en = b.cstart[c + 1];
    int r = 0;
    int u = st;
    for (; u + 4 <= en; u += 4) {
        const int a0 = b.tsc[u], a1 = b.tsc[u + 1], a2 = b.tsc[u + 2], a3 = b.tsc[u + 3];
        r += (a0 < t) + (a1 < t) + (a2 < t) + (a3 < t);
    }
    for (; u < en; ++u) r += (b.tsc[u] < t);
    const int64_t nw = st + r;
    b.x[parity][nw] = p;
    const int4 q = quantize4(g, p.x, p.y, p.z, p.w);
    b.xq[parity][nw] = q;
    if (g.x3_on) store_q3(b.x3[parity], nw, q);
    b.xb[nw] = p.x;
    b.xb[n + nw] = p.y;
    b.xb[2 * n + nw] = p.z;
    for (int d = 0; d < 3; ++d) {
        b.v[d * n + nw] = vv[d];
        b.img[d * n + nw] = im[d];
    }
    b.tag[nw] = t;
    // the inverse permutation serves only the bonded remap of the list
    // build, which also copies the per-particle bond and angle counts
    if (bonded) b.inv[t] = (int32_t)nw;
}

__global__ void __launch_bounds__(kBlock) k_rank(Geom g, Bufs b, int parity, int bonded) {
    if (!rebuild_requested(b, parity)) return;
    for (int64_t s = gtid(); s < g.n; s += gstride()) rank_one(g, b, s, parity, bonded);
}

// The whole sort of a small system by one block: counts and cursors in LDS,
// the passes separated by block barriers.  A step that rebuilds nothing then
// launches one kernel for the sort instead of four (each launch that returns
// costs 1.5-2.9 us), and one that does pays no launch gaps.
constexpr int kSmallSort = 4096;    // particles
constexpr int kSmallCells = 8192;   // cells (32 KB of LDS)
constexpr int kSmallBlock = 1024;
__global__ void __launch_bounds__(kSmallBlock) k_sort_small(Geom g, Bufs b, int parity, int bonded, int advance) {
    __shared__ int cnt[kSmallCells];
    __shared__ int wsum[kSmallBlock / 64];
    if (advance && threadIdx.x == 0) advance_step(b, parity);
    if (!rebuild_requested(b, parity)) return;
    const int n = (int)g.n, ncell = (int)g.ncell, tid = threadIdx.x;
    for (int c = tid; c < ncell; c += kSmallBlock) cnt[c] = 0;
    __syncthreads();
    for (int i = tid; i < n; i += kSmallBlock) {
        const uint32_t c = cell_of(g, b.x[parity][i]);
        b.cellid[i] = c;
        atomicAdd(&cnt[c], 1);
    }
    __syncthreads();
    // exclusive scan, a run of consecutive cells per thread
    const int per = (ncell + kSmallBlock - 1) / kSmallBlock;
    const int c0 = min(tid * per, ncell), c1 = min(c0 + per, ncell);
    int sum = 0;
    for (int c = c0; c < c1; ++c) sum += cnt[c];
    int x = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o, 64);
        if ((tid & 63) >= o) x += y;
    }
    if ((tid & 63) == 63) wsum[tid >> 6] = x;
    __syncthreads();
    int e = x - sum;
    for (int w = 0; w < (tid >> 6); ++w) e += wsum[w];
    for (int c = c0; c < c1; ++c) {
        const int k = cnt[c];
        cnt[c] = e;
        b.cstart[c] = e;
        e += k;
    }
    if (tid == 0) b.cstart[ncell] = n;
    __syncthreads();
    for (int i = tid; i < n; i += kSmallBlock) {
        const double4 p = b.x[parity][i];
        double vv[3];
        int32_t im[3];
        for (int d = 0; d < 3; ++d) {
            vv[d] = b.v[(int64_t)d * n + i];
            im[d] = b.img[(int64_t)d * n + i];
        }
        const int slot = atomicAdd(&cnt[b.cellid[i]], 1);
        stash(b, n, slot, p, vv, im, b.tag[i]);
    }
    __syncthreads();
    for (int s = tid; s < n; s += kSmallBlock) rank_one(g, b, s, parity, bonded);
}

// ------------------------------------------------------------------ rebuild: Verlet list

// r_ij^2 in FP64 with the operation order of the plain definition
// ((dx*dx + dy*dy) + dz*dz, no fused multiply-add): the list and cutoff
// decisions taken with it equal those of any implementation doing the same
// IEEE operations on the same positions.
__device__ __forceinline__ double exact_r2(const Geom& g, const double4& a, const double4& b) {
#pragma clang fp contract(off)
    const double dx = mimg(b.x - a.x, g.L[0], g.invL[0]);
    const double dy = mimg(b.y - a.y, g.L[1], g.invL[1]);
    const double dz = mimg(b.z - a.z, g.L[2], g.invL[2]);
    return (dx * dx + dy * dy) + dz * dz;
}

// distance along one axis from a point at offset u inside its cell to the
// cell o cells away
__device__ __forceinline__ float cell_gap(int o, float u, float h) {
    float d = o > 0 ? (float)o * h - u : (o < 0 ? u + (float)(-o - 1) * h : 0.0f);
    return d > 0.0f ? d : 0.0f;
}

__device__ __forceinline__ int wrapc(int c, int nc) { return c < 0 ? c + nc : (c >= nc ? c - nc : c); }

// Bond and angle counts and partners of sorted particle i, partners from
// tags to sorted indices.
__device__ __forceinline__ void remap_bonded(const Bufs& b, int64_t n, int64_t i) {
    const int32_t t = b.tag[i];
    const int tc = b.tcnt_t[t];
    b.tcnt_s[i] = tc;
    const int nb = tc & 0xff, na = tc >> 8;
    for (int k = 0; k < nb; ++k) b.bp_s[(int64_t)k * n + i] = b.inv[b.bp_t[(int64_t)k * n + t]];
    for (int k = 0; k < na; ++k) {
        const int2 e = b.ang_t[(int64_t)k * n + t];
        const int role = (int)((uint32_t)e.x >> 30);
        const int o1 = e.x & 0x3fffffff;
        b.ang_s[(int64_t)k * n + i] = make_int2(b.inv[o1] | (role << 30), b.inv[e.y]);
    }
}

// NL(i) = { j != i : r_ij^2 < rv^2 } over the cells within rv of particle i
// (stencil of (2kc+1)^3 cells of side >= rv/kc, cells farther than rv
// skipped).  The test runs on the fixed-point positions and is retaken in
// FP64 (exact_r2) inside a band around rv that bounds the fixed-point
// rounding, so the sets are those of the FP64 definition.  Row order:
// stencil (z, y, x offsets), then sorted index.  Also remaps the bonded
// topology from tags to sorted indices.
constexpr int kNlLds = 24;  // row slots staged in LDS by the per-particle build (25 KB per block with the spare row)

// Store a group of four tested candidates j0..j0+3 (hits flagged in `in`) to
// a per-particle row: its first kNlLds slots in LDS (buf, [slot][lane] of the
// wavefront, row kNlLds a spare), the rest in the list.  While the next four
// slots lie in LDS every candidate is stored, a miss to the spare row, with
// no branch; past them (LIST_PATH) one masked store per hit; otherwise, and
// for the group that crosses from LDS to the list, the general path.  Hits
// beyond the capacity are counted, not stored.  The list-only path pays where
// rows run well past the LDS slots (dense fluids on half cells or by flag);
// where rows end near them (the sheared DPD fluid, ~28 slots) the lanes split
// over three paths and it cost 11 % of the build, so that build leaves it out.
template <bool LIST_PATH>
__device__ __forceinline__ void nl_store4(int32_t (*buf)[64], int ln, int32_t* __restrict__ nlrow, int cap,
                                          const bool (&in)[4], int j0, int& cnt) {
    if (cnt + 4 <= kNlLds) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            buf[in[u] ? cnt : kNlLds][ln] = j0 + u;
            cnt += in[u] ? 1 : 0;
        }
    } else if (LIST_PATH && cnt >= kNlLds) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (in[u] & (cnt < cap)) nlrow[nl_off(cnt)] = j0 + u;
            cnt += in[u] ? 1 : 0;
        }
    } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (in[u]) {
                if (cnt < cap) {
                    if (cnt < kNlLds) buf[cnt][ln] = j0 + u;
                    else nlrow[nl_off(cnt)] = j0 + u;
                }
                ++cnt;
            }
        }
    }
}
// nlbuf: kNlLds + 1 rows of the wavefront's LDS.
__device__ __forceinline__ void nl_one(const Geom& g, const Bufs& b, int64_t i, int parity, int bonded,
                                       int32_t (*nlbuf)[64], int& local_max, bool& overflow) {
    const int64_t n = g.n;
    const double4* __restrict__ x = b.x[parity];
    const int4* __restrict__ xq = b.xq[parity];
    const float hy = (float)g.h[1], hz = (float)g.h[2];
    const int kc = g.kc;
    {
        const double4 xi = x[i];
        const int4 qi = xq[i];
        int cx, cy, cz;
        cell_coords(g, xi.x, xi.y, xi.z, cx, cy, cz);
        const float uy = (float)(xi.y - cy * g.h[1]);
        const float uz = (float)(xi.z - cz * g.h[2]);
        int cnt = 0;
        const int self = (int)i;
        int32_t* __restrict__ nlrow = b.nl + nl_base(i, g.cap);
        // The first kNlLds slots of each row collect in LDS, [slot][lane] per
        // wavefront, and leave in whole-wavefront stores at the end: the
        // hits of the lanes fall in different iterations, so direct stores
        // would cost one partly masked store instruction per hit event.
        // Row kNlLds is a spare that takes the stores of candidates that miss.
        const int ln = threadIdx.x & 63;
        auto put = [&](int k, int j) {
            if (k < kNlLds) nlbuf[k][ln] = j;
            else nlrow[nl_off(k)] = j;
        };
        // Cells cx-kc .. cx+kc of one (y, z) row are consecutive in the cell
        // order, so their particles form one contiguous range of the sorted
        // arrays (two when the row wraps around the box).  Candidates are
        // gathered four at a time, the last one repeated past the end of the
        // range, so a short range costs one memory round trip.  The four
        // tests become flags with one branch for the rare FP64 band, and the
        // stores take as few branches as the row's position allows
        // (nl_store4): per-candidate branches cost more scalar and branch
        // issue than the tests themselves.
        auto test_range = [&](int st, int en) {
            for (int j = st; j < en; j += 4) {
                int4 qq[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) qq[u] = xq[min(j + u, en - 1)];
                bool in[4], band[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float dx = qdiff(qq[u].x, qi.x, g.ql[0]);
                    const float dy = qdiff(qq[u].y, qi.y, g.ql[1]);
                    const float dz = qdiff(qq[u].z, qi.z, g.ql[2]);
                    const float r2 = dx * dx + dy * dy + dz * dz;
                    // bitwise, not short-circuit: no branch around the test
                    const bool ok = (j + u < en) & (j + u != self);
                    in[u] = ok & (r2 < g.rv2lo);
                    band[u] = ok & (r2 >= g.rv2lo) & (r2 < g.rv2hi);
                }
                if (band[0] | band[1] | band[2] | band[3]) {
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (band[u]) in[u] = exact_r2(g, xi, x[j + u]) < g.rv2;
                }
                nl_store4<true>(nlbuf, ln, nlrow, g.cap, in, j, cnt);
            }
        };
        const int xlo = cx - kc, xhi = cx + kc;   // inclusive cell range along x
        const int nx = g.nc[0];
        const bool wl = xlo < 0, wh = xhi >= nx;
        const int side = 2 * kc + 1, nv = 2 * side * side;
        const int32_t* __restrict__ cs = b.cstart;
        // Piece v is the first or second range of stencil row v / 2 (rows
        // z-major, empty when the row is out of reach or does not wrap).  The
        // cell bounds of piece v + 1 are loaded before the candidates of
        // piece v are tested, so the two loads overlap.
        auto piece = [&](int v, int& a, int& e) {
            a = e = 0;
            const int r = v >> 1, pc = v & 1;
            const int oz = r / side - kc, oy = r % side - kc;
            const float gz = cell_gap(oz, uz, hz);
            const float gz2 = gz * gz;
            if (gz2 > g.rv2hi) return;
            const float gy = cell_gap(oy, uy, hy);
            if (gz2 + gy * gy > g.rv2hi) return;
            const int nz = wrapc(cz + oz, g.nc[2]), ny = wrapc(cy + oy, g.nc[1]);
            const int64_t rowc = ((int64_t)nz * g.nc[1] + ny) * nx;
            if (!wl && !wh) {
                if (pc == 0) { a = cs[rowc + xlo]; e = cs[rowc + xhi + 1]; }
            } else if (wl) {
                if (pc == 0) { a = cs[rowc + nx + xlo]; e = cs[rowc + nx]; }
                else { a = cs[rowc]; e = cs[rowc + xhi + 1]; }
            } else {
                if (pc == 0) { a = cs[rowc + xlo]; e = cs[rowc + nx]; }
                else { a = cs[rowc]; e = cs[rowc + xhi - nx + 1]; }
            }
        };
        int pa, pe;
        piece(0, pa, pe);
        for (int v = 0; v < nv; ++v) {
            int na = 0, ne = 0;
            if (v + 1 < nv) piece(v + 1, na, ne);
            test_range(pa, pe);
            pa = na;
            pe = ne;
        }
        b.ncount[i] = cnt;
        if (cnt > local_max) local_max = cnt;
        if (cnt > g.cap) overflow = true;
        // pad the row to a multiple of 8 with the particle itself (r = 0,
        // never inside a cutoff) so that step kernels stream whole batches
        const int nslot = min(((cnt + 7) & ~7), g.cap);
        for (int k = cnt; k < nslot; ++k) put(k, (int)i);
#pragma unroll
        for (int k = 0; k < kNlLds; ++k)
            if (k < nslot) nlrow[nl_off(k)] = nlbuf[k][ln];
        if (bonded) remap_bonded(b, n, i);
    }
}

// Longest row and overflow flag.  Atomics on one address serialize (tens of
// ns each, measured), so a wavefront raises the maximum only when its own
// row is longer than the value it reads; a stale read costs one redundant
// atomic, never a wrong maximum.
__device__ __forceinline__ void nl_epilogue(const Bufs& b, int local_max, bool overflow) {
    for (int o = 32; o >= 1; o >>= 1) {
        const int y = __shfl_xor(local_max, o, 64);
        local_max = y > local_max ? y : local_max;
    }
    if ((threadIdx.x & 63) == 0 && local_max > 0) {
        const int cur = __hip_atomic_load(&b.ctl->nl_max, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (local_max > cur) atomicMax(&b.ctl->nl_max, local_max);
    }
    if (__any(overflow) && (threadIdx.x & 63) == 0) atomicOr(&b.ctl->status, MD_FLAG_NL_OVERFLOW);
}

__global__ void __launch_bounds__(kBlock) k_nl_build(Geom g, Bufs b, int parity, int bonded) {
    __shared__ int32_t nlbuf[kBlock / 64][kNlLds + 1][64];
    if (!rebuild_requested(b, parity)) return;
    int local_max = 0;
    bool overflow = false;
    for (int64_t i = gtid_xcd(); i < g.n; i += gstride())
        nl_one(g, b, i, parity, bonded, nlbuf[threadIdx.x >> 6], local_max, overflow);
    nl_epilogue(b, local_max, overflow);
}

// The same lists, one wavefront per particle, for systems whose particles
// leave the GPU idle one per lane: the particle's stencil ranges are bounded by
// one lane each, their candidates tested 64 at a time and the hits compacted by
// ballot, so a row takes a few memory round trips instead of one per stencil
// row and candidate group.  Row order and decisions as nl_one.
__global__ void __launch_bounds__(kBlock) k_nl_wave(Geom g, Bufs b, int parity, int bonded) {
    if (!rebuild_requested(b, parity)) return;
    const int lane = threadIdx.x & 63;
    const int64_t n = g.n;
    const int i = (int)((int64_t)blockIdx.x * (kBlock / 64)) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64));
    if (i >= n) return;
    const double4* __restrict__ x = b.x[parity];
    const int4* __restrict__ xq = b.xq[parity];
    const double4 xi = x[i];
    const int4 qi = xq[i];
    int cx, cy, cz;
    cell_coords(g, xi.x, xi.y, xi.z, cx, cy, cz);
    const int kc = g.kc, nx = g.nc[0], side = 2 * kc + 1, cap = g.cap;
    // lane v: the first or second contiguous range of stencil row v / 2
    int pa = 0, len = 0;
    if (lane < 2 * side * side) {
        const int r = lane >> 1, pc = lane & 1, oz = r / side - kc, oy = r % side - kc;
        const float gz = cell_gap(oz, (float)(xi.z - cz * g.h[2]), (float)g.h[2]);
        const float gy = cell_gap(oy, (float)(xi.y - cy * g.h[1]), (float)g.h[1]);
        if (gz * gz + gy * gy <= g.rv2hi) {
            const int nz = wrapc(cz + oz, g.nc[2]), ny = wrapc(cy + oy, g.nc[1]);
            const int64_t rowc = ((int64_t)nz * g.nc[1] + ny) * nx;
            const int l = wrapc(cx - kc, nx), h = l + 2 * kc;
            int e = 0;
            if (h < nx) {
                if (pc == 0) { pa = b.cstart[rowc + l]; e = b.cstart[rowc + h + 1]; }
            } else if (pc == 0) {
                pa = b.cstart[rowc + l]; e = b.cstart[rowc + nx];
            } else {
                pa = b.cstart[rowc]; e = b.cstart[rowc + h - nx + 1];
            }
            len = e - pa;
        }
    }
    int end = len;      // prefix of the candidates up to this range
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(end, o, 64);
        if (lane >= o) end += y;
    }
    const int total = __builtin_amdgcn_readlane(end, 63);
    uint64_t todo = __ballot(len > 0);
    int32_t* __restrict__ nlrow = b.nl + nl_base(i, cap);
    int cnt = 0;
    for (int c0 = 0; c0 < total; c0 += 64) {
        // candidate c0 + lane: the range that holds it
        int j = i;
        uint64_t rest = todo;
        while (rest) {
            const int v = __ffsll((unsigned long long)rest) - 1;
            rest &= rest - 1;
            const int hi = __builtin_amdgcn_readlane(end, v), lo = hi - __builtin_amdgcn_readlane(len, v);
            if (lo >= c0 + 64) break;
            if (hi <= c0 + 64) todo &= ~(1ull << v);    // ends in this chunk
            const int c = c0 + lane;
            if (c >= lo && c < hi) j = __builtin_amdgcn_readlane(pa, v) + c - lo;
        }
        const int4 q = xq[j];
        const float dx = qdiff(q.x, qi.x, g.ql[0]), dy = qdiff(q.y, qi.y, g.ql[1]), dz = qdiff(q.z, qi.z, g.ql[2]);
        const float r2 = dx * dx + dy * dy + dz * dz;
        bool in = j != i && r2 < g.rv2lo;
        if (j != i && r2 >= g.rv2lo && r2 < g.rv2hi) in = exact_r2(g, xi, x[j]) < g.rv2;
        const uint64_t m = __ballot(in);
        const int pos = cnt + (int)__popcll(m & ((1ull << lane) - 1));
        if (in && pos < cap) nlrow[nl_off(pos)] = j;
        cnt += (int)__popcll(m);
    }
    if (lane == 0) b.ncount[i] = cnt;
    const int k = cnt + lane;   // padding to a multiple of 8 with the particle itself
    if (k < ((cnt + 7) & ~7) && k < cap) nlrow[nl_off(k)] = i;
    if (bonded) {
        // remap_bonded, a lane per bond and angle
        const int32_t t = b.tag[i];
        const int tc = b.tcnt_t[t];
        if (lane == 0) b.tcnt_s[i] = tc;
        if (lane < (tc & 0xff)) b.bp_s[(int64_t)lane * n + i] = b.inv[b.bp_t[(int64_t)lane * n + t]];
        const int a = lane - 32;
        if (a >= 0 && a < (tc >> 8)) {
            const int2 e = b.ang_t[(int64_t)a * n + t];
            const int role = (int)((uint32_t)e.x >> 30);
            b.ang_s[(int64_t)a * n + i] = make_int2(b.inv[e.x & 0x3fffffff] | (role << 30), b.inv[e.y]);
        }
    }
    nl_epilogue(b, cnt, cnt > cap);
}

// ------------------------------------------------------------------ Lees-Edwards shear
//
// Flow along x, gradient along y (section "New Features": Lees-Edwards
// boundary conditions).  The image one box above is displaced by
// delta(step) = fmod(shear_rate Ly (step dt), Lx) and moves with
// +shear_rate Ly along x.  Minimum image of d = r_j - r_i: dy by
// compare-and-shift, s = +1 when dy > Ly/2 (j's nearest image lies one box
// below: x_j - delta), -1 when dy < -Ly/2; dx = the x minimum image of
// x_j - x_i, then for s != 0 the x minimum image of dx - s delta_w
// (delta_w = delta folded into (-Lx/2, Lx/2]).  FP64 operations in that
// order, so list and cutoff decisions equal any implementation doing the
// same operations.

__device__ __forceinline__ double le_delta(const Geom& g, int64_t step) {
    double d = fmod(g.le_rate_Ly * ((double)step * g.le_dt), g.L[0]);
    return d < 0.0 ? d + g.L[0] : d;
}
__device__ __forceinline__ double le_fold(const Geom& g, double d) { return d > g.hL[0] ? d - g.L[0] : d; }

__device__ __forceinline__ double exact_r2_le(const Geom& g, const double4& a, const double4& b, double dw) {
#pragma clang fp contract(off)
    double dy = b.y - a.y;
    int sy = 0;
    if (dy > g.hL[1]) { dy -= g.L[1]; sy = 1; }
    else if (dy < -g.hL[1]) { dy += g.L[1]; sy = -1; }
    double dx = mimg(b.x - a.x, g.L[0], g.invL[0]);
    if (sy != 0) dx = mimg(dx - sy * dw, g.L[0], g.invL[0]);
    const double dz = mimg(b.z - a.z, g.L[2], g.invL[2]);
    return (dx * dx + dy * dy) + dz * dz;
}

// Sign s of the sheared image from the fixed-point y coordinates: the raw
// difference beyond half the box (2^31 units).
__device__ __forceinline__ int le_sign_q(uint32_t qiy, uint32_t qjy) {
    const int64_t d = (int64_t)qjy - (int64_t)qiy;
    return d > 0x80000000LL ? 1 : (d < -0x80000000LL ? -1 : 0);
}

// Fixed-point differences r_j - r_i under the shear (qd = the offset delta in
// units of Lx 2^-32); s as above.
struct DiffLEQ {
    float l0, l1, l2;
    uint32_t qd;
    __device__ int operator()(const int4& a, const int4& b, float& dx, float& dy, float& dz) const {
        const int s = le_sign_q((uint32_t)a.y, (uint32_t)b.y);
        dx = (float)(int32_t)((uint32_t)b.x - (uint32_t)a.x - (uint32_t)(s * (int64_t)qd)) * l0;
        dy = qdiff(b.y, a.y, l1);
        dz = qdiff(b.z, a.z, l2);
        return s;
    }
};

// NL(i) under the shear, one particle per lane: as nl_one, except that a
// stencil row reached across the y boundary (s != 0) scans the x cells
// around x_i + s delta (one cell of margin each side, the whole row when that
// covers it).  Rows are in stencil order; sets equal the FP64 definition.
__device__ __forceinline__ void nl_one_le(const Geom& g, const Bufs& b, int64_t i, int parity, int bonded,
                                          double delta, double dw, uint32_t qd, int& local_max, bool& overflow) {
    const int64_t n = g.n;
    const double4* __restrict__ x = b.x[parity];
    const int4* __restrict__ xq = b.xq[parity];
    const int kc = g.kc, nx = g.nc[0];
    const double4 xi = x[i];
    const int4 qi = xq[i];
    int cx, cy, cz;
    cell_coords(g, xi.x, xi.y, xi.z, cx, cy, cz);
    const float uy = (float)(xi.y - cy * g.h[1]);
    const float uz = (float)(xi.z - cz * g.h[2]);
    const DiffLEQ df{g.ql[0], g.ql[1], g.ql[2], qd};
    int32_t* __restrict__ nlrow = b.nl + nl_base(i, g.cap);
    int cnt = 0;
    // the first kNlLds slots collect in LDS, [slot][lane] per wavefront, and
    // leave in whole-wavefront stores at the end (as in the plain build)
    // (row kNlLds is the spare of the misses, as there)
    __shared__ int32_t nlbuf_le[kBlock / 64][kNlLds + 1][64];
    const int wv = threadIdx.x >> 6, ln = threadIdx.x & 63;
    const int self = (int)i;
    auto put = [&](int k, int j) {
        if (k < kNlLds) nlbuf_le[wv][k][ln] = j;
        else nlrow[nl_off(k)] = j;
    };
    // candidates gathered four at a time, the last one repeated past the end
    // of the range; tests as flags and stores as in the plain build
    auto test_range = [&](int st, int en) {
        for (int j0 = st; j0 < en; j0 += 4) {
            int4 qq[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) qq[u] = xq[min(j0 + u, en - 1)];
            bool in[4], band[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                float dx, dy, dz;
                df(qi, qq[u], dx, dy, dz);
                const float r2 = dx * dx + dy * dy + dz * dz;
                const bool ok = (j0 + u < en) & (j0 + u != self);
                in[u] = ok & (r2 < g.rv2lo);
                band[u] = ok & (r2 >= g.rv2lo) & (r2 < g.rv2hi);
            }
            if (band[0] | band[1] | band[2] | band[3]) {
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (band[u]) in[u] = exact_r2_le(g, xi, x[j0 + u], dw) < g.rv2;
            }
            nl_store4<false>(nlbuf_le[wv], ln, nlrow, g.cap, in, j0, cnt);
        }
    };
    // Piece v is the first or second contiguous range of stencil row v / 2
    // (rows z-major; empty when the row is out of reach or does not wrap).
    // Across the y-boundary the row's x-range is re-centred on x_i +- delta
    // with one cell of margin each side (the whole row when that covers it).
    // The bounds of piece v + 1 are loaded before piece v is tested.
    const int32_t* __restrict__ cs = b.cstart;
    const int side = 2 * kc + 1, nv = 2 * side * side;
    const double rv = sqrt(g.rv2);
    auto piece = [&](int v, int& a, int& e) {
        a = e = 0;
        const int r = v >> 1, pc = v & 1;
        const int oz = r / side - kc, oy = r % side - kc;
        const float gz = cell_gap(oz, uz, (float)g.h[2]);
        if (gz * gz > g.rv2hi) return;
        const float gy = cell_gap(oy, uy, (float)g.h[1]);
        if (gz * gz + gy * gy > g.rv2hi) return;
        const int nz = wrapc(cz + oz, g.nc[2]);
        const int yraw = cy + oy;
        const int sh = yraw < 0 ? 1 : (yraw >= g.nc[1] ? -1 : 0);
        const int ny = wrapc(yraw, g.nc[1]);
        const int64_t rowc = ((int64_t)nz * g.nc[1] + ny) * nx;
        int lo = cx - kc, hi = cx + kc;
        if (sh != 0) {
            const double c0 = xi.x + sh * delta;
            lo = (int)floor((c0 - rv) * g.invh[0]) - 1;
            hi = (int)floor((c0 + rv) * g.invh[0]) + 1;
        }
        if (hi - lo + 1 >= nx) {
            if (pc == 0) { a = cs[rowc]; e = cs[rowc + nx]; }
            return;
        }
        // [lo, hi] modulo nx: one or two contiguous ranges of cells
        const int l = ((lo % nx) + nx) % nx;
        const int h = l + (hi - lo);
        if (h < nx) {
            if (pc == 0) { a = cs[rowc + l]; e = cs[rowc + h + 1]; }
        } else if (pc == 0) {
            a = cs[rowc + l]; e = cs[rowc + nx];
        } else {
            a = cs[rowc]; e = cs[rowc + h - nx + 1];
        }
    };
    int pa, pe;
    piece(0, pa, pe);
    for (int v = 0; v < nv; ++v) {
        int na = 0, ne = 0;
        if (v + 1 < nv) piece(v + 1, na, ne);
        test_range(pa, pe);
        pa = na;
        pe = ne;
    }
    b.ncount[i] = cnt;
    if (cnt > local_max) local_max = cnt;
    if (cnt > g.cap) overflow = true;
    const int nslot = min(((cnt + 7) & ~7), g.cap);
    for (int k = cnt; k < nslot; ++k) put(k, (int)i);
#pragma unroll
    for (int k = 0; k < kNlLds; ++k)
        if (k < nslot) nlrow[nl_off(k)] = nlbuf_le[wv][k][ln];
    if (bonded) remap_bonded(b, n, i);
}

__global__ void __launch_bounds__(kBlock) k_nl_build_le(Geom g, Bufs b, int parity, int bonded) {
    if (!rebuild_requested(b, parity)) return;
    const double delta = le_delta(g, b.ctl->step);
    const double dw = le_fold(g, delta);
    const uint32_t qd = quantize(delta, g.qs[0]);
    int local_max = 0;
    bool overflow = false;
    for (int64_t i = gtid_xcd(); i < g.n; i += gstride())
        nl_one_le(g, b, i, parity, bonded, delta, dw, qd, local_max, overflow);
    nl_epilogue(b, local_max, overflow);
}

// ------------------------------------------------------------------ list build on the matrix cores
//
// The lists of nl_one, entry for entry, and the sets of nl_one_le (under shear
// a segment's range may cover a whole row where a lane's own does not, and the
// row then starts elsewhere), built one wavefront per 64-particle tile of the
// sorted order (the tile of the list layout).  The tile's particles lie in a few consecutive cells; lanes of one (y, z) cell row
// form a segment whose x-cells span [x0, x1].  The segment's candidates are
// the particles of cells [x0 - kc, x1 + kc] in each of the (2kc+1)^2
// neighbouring rows, in nl_one's order (rows z-major, a wrapped x-range high
// part first, sorted index), taken 32 at a time over the ends of the ranges.
// A candidate outside a lane's own stencil is at least kc cell sides >= rv
// away and never passes the test, and a lane's own candidates keep their
// relative order.
//
// The squared distances of 32 candidates to the tile's 64 particles are a
// contraction of length 4, (x, y, z, |r_j|^2) . (-2x, -2y, -2z, 1), on
// coordinates relative to the segment's centre: four
// v_mfma_f32_32x32x2_f32 with |r_i|^2 - rv^2 as the accumulator's start, so
// that the sign bit of the result is the list test.  One v_alignbit per result
// collects the sign bits, one v_min3 per two results the distance to the
// threshold; a chunk that comes within the rounding bound of it (nl_delta) is
// retaken in FP64 for the candidates concerned, so the sets are those of the
// FP64 definition.  Coordinates relative to the centre are the minimum image
// only where half the segment and rv together stay below half the box: a
// segment spans at most nx - 2kc - 1 cells, and the build needs 2kc + 2 cells
// per side (Geom::nl_mat).
//
// The hits of 32 candidates are one 32-bit word per lane.  Each lane queues
// its words with hits in LDS (W of them), then all lanes write their rows
// together, slot by slot, as whole 256-byte stores.  Writing each hit when it
// is found cost the texture path 625 partly masked stores per tile and sent
// the list through the L2 4.2 times (1.44 GB for 344 MB at 1M particles).
typedef float f32x16 __attribute__((ext_vector_type(16)));
constexpr int kNlSpan = 31;     // x-cells of a segment beyond its first: bounds the coordinates, so the rounding
// Words a lane queues before the rows are written: 18 let 16 wavefronts share
// a CU's LDS, as many as the registers allow.  A particle of a dense fluid (19
// per cell) has hits in 20-30 words; 23 words (12 wavefronts) took 363 us per
// 1M-particle build, 14 words 344, 18 words 326.
constexpr int kNlWords = 18;

struct NlWave {
    uint2 q[kNlWords + 1][64];  // queued (hit word, candidate of its bit 0), [position][lane]
};

// Offsets of a sheared system at its build step (zeros otherwise).
struct LeNl {
    double delta, dw;
    uint32_t qd;
};

// Lanes' (lower half of a, lower half of b) and (upper half of a, upper half
// of b): the two 32-particle blocks' operands from per-lane values.
__device__ __forceinline__ void half_swap(uint32_t& a, uint32_t& b) {
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}
__device__ __forceinline__ void half_swap(float& a, float& b) {
    uint32_t u = __float_as_uint(a), v = __float_as_uint(b);
    half_swap(u, v);
    a = __uint_as_float(u);
    b = __uint_as_float(v);
}

// Bits e = 0..15 set where d[e] is negative.
__device__ __forceinline__ uint32_t sign_bits(const f32x16& d) {
    uint32_t m = 0;
#pragma unroll
    for (int e = 15; e >= 0; --e) m = __builtin_amdgcn_alignbit(m, __float_as_uint(d[e]), 31);
    return m;
}

// v0, v1 or v2 for a position below e0, below e1 or past it (by value: a
// conditional over struct members selects an address and puts the struct in
// scratch memory).
__device__ __forceinline__ int pick(int k, int e0, int e1, int v0, int v1, int v2) {
    const int v = k < e1 ? v1 : v2;
    return k < e0 ? v0 : v;
}

template <bool LE>
__device__ __forceinline__ void nl_mtile(const Geom& g, const Bufs& b, int64_t t, int parity, int bonded, NlWave& sh,
                                         const LeNl& le, int& local_max, bool& overflow) {
    const int lane = threadIdx.x & (kTile - 1);
    const int64_t n = g.n, p0 = t * kTile;
    const int self = (int)p0 + lane;
    const int nv = n - p0 < kTile ? (int)(n - p0) : kTile;
    const bool valid = lane < nv;
    const double4* __restrict__ x = b.x[parity];
    const char* __restrict__ xqb = reinterpret_cast<const char*>(b.xq[parity]);
    const int32_t* __restrict__ cs = b.cstart;
    const int kc = g.kc, nx = g.nc[0], cap = g.cap;
    int cxl = -1, cyl = -1, czl = -1;
    int4 qi = make_int4(0, 0, 0, 0);
    if (valid) {
        const double4 xi = x[self];
        cell_coords(g, xi.x, xi.y, xi.z, cxl, cyl, czl);
        qi = b.xq[parity][self];
    }
    char* const rowb = reinterpret_cast<char*>(b.nl + p0 * cap) + 4 * lane;
    int cnt = 0;
    // the candidate (of 64) a lane loads: matrix row 8 (e / 4) + 4 h + e % 4
    // of a 32-candidate half comes back as bit 16 h + e of its hit word
    const int ck = (lane & 32) + ((lane >> 2) & 1) * 16 + ((lane & 31) >> 3) * 4 + (lane & 3);
    const float l0 = g.ql[0], l1 = g.ql[1], l2 = g.ql[2];
    const int xlimit = min(nx - 2 * kc - 2, kNlSpan);
    int lo = 0;
    while (lo < nv) {
        const int x0 = __builtin_amdgcn_readlane(cxl, lo);
        const int y0 = __builtin_amdgcn_readlane(cyl, lo);
        const int z0 = __builtin_amdgcn_readlane(czl, lo);
        const int hi = lo + (int)__popcll(__ballot(valid && lane >= lo && cyl == y0 && czl == z0 && cxl <= x0 + xlimit));
        const int x1 = __builtin_amdgcn_readlane(cxl, hi - 1);
        const bool mine = lane >= lo && lane < hi;
        // lane v: the first or second contiguous range of stencil row v / 2
        // (rows z-major; empty when the row does not wrap)
        const int side = 2 * kc + 1;
        int pa = 0, pe = 0, psg = 0;
        if (lane < 2 * side * side) {
            const int r = lane >> 1, pc = lane & 1;
            const int nz = wrapc(z0 + r / side - kc, g.nc[2]);
            const int yraw = y0 + r % side - kc, ny = wrapc(yraw, g.nc[1]);
            const int64_t rowc = ((int64_t)nz * g.nc[1] + ny) * nx;
            int xa = x0 - kc, xb = x1 + kc;
            if (LE) {
                // across the y-boundary the x-range is re-centred by the
                // offset, with one cell of margin each side
                psg = yraw < 0 ? 1 : (yraw >= g.nc[1] ? -1 : 0);
                if (psg != 0) {
                    const double rv = sqrt(g.rv2), sd = psg * le.delta;
                    xa = (int)floor((x0 * g.h[0] + sd - rv) * g.invh[0]) - 1;
                    xb = (int)floor(((x1 + 1) * g.h[0] + sd + rv) * g.invh[0]) + 1;
                }
            }
            if (LE && xb - xa + 1 >= nx) {
                if (pc == 0) { pa = cs[rowc]; pe = cs[rowc + nx]; }
            } else {
                const int l = LE ? ((xa % nx) + nx) % nx : wrapc(xa, nx);
                const int h = l + (xb - xa);
                if (h < nx) {
                    if (pc == 0) { pa = cs[rowc + l]; pe = cs[rowc + h + 1]; }
                } else if (pc == 0) {
                    pa = cs[rowc + l]; pe = cs[rowc + nx];
                } else {
                    pa = cs[rowc]; pe = cs[rowc + h - nx + 1];
                }
            }
        }
        uint64_t pm = __ballot(pe > pa);
        // coordinates relative to the segment's centre, the particles' operands
        const uint32_t ox = (uint32_t)__builtin_amdgcn_readfirstlane((int)quantize(0.5 * (x0 + x1 + 1) * g.h[0], g.qs[0]));
        const uint32_t oy = (uint32_t)__builtin_amdgcn_readfirstlane((int)quantize((y0 + 0.5) * g.h[1], g.qs[1]));
        const uint32_t oz = (uint32_t)__builtin_amdgcn_readfirstlane((int)quantize((z0 + 0.5) * g.h[2], g.qs[2]));
        float bx0, bx1, bz0, bz1, c0, c1;
        {
            const float fx = qdiff((uint32_t)qi.x, ox, l0), fy = qdiff((uint32_t)qi.y, oy, l1),
                        fz = qdiff((uint32_t)qi.z, oz, l2);
            bx0 = -2.f * fx; bx1 = -2.f * fy;
            half_swap(bx0, bx1);
            bz0 = -2.f * fz; bz1 = 1.f;
            half_swap(bz0, bz1);
            c0 = c1 = fx * fx + fy * fy + fz * fz - (float)g.rv2;
            half_swap(c0, c1);
        }
        f32x16 C0, C1;
#pragma unroll
        for (int e = 0; e < 16; ++e) { C0[e] = c0; C1[e] = c1; }
        // Rounding bound of a result near the threshold, where every
        // coordinate is within half the segment plus the stencil of the
        // centre: with E the length of that corner vector, coordinates are
        // within 2^-23 relative (8 units of 2^-24 E^2 in r^2), |r_i|^2 and
        // |r_j|^2 within 3 units each, the accumulator's start within 1, the
        // four products and sums within 24; 64 units, and the fixed-point
        // band.
        float delta;
        {
            const float ex = (0.5f * (float)(x1 - x0 + 1) + (float)kc) * (float)g.h[0];
            const float ey = (0.5f + (float)kc) * (float)g.h[1], ez = (0.5f + (float)kc) * (float)g.h[2];
            delta = 64.f * 0x1.0p-24f * (ex * ex + ey * ey + ez * ez) + (g.rv2hi - (float)g.rv2);
        }
        int qn = 0;         // words queued by this lane
        // every lane writes its next hit, slot by slot; the word after the
        // current one is read ahead, an empty word ends the queue
        auto emit = [&]() __attribute__((always_inline)) {
            sh.q[qn][lane] = make_uint2(0u, 0u);
            __builtin_amdgcn_wave_barrier();
            uint2 c = sh.q[0][lane];
            int k = min(1, qn);
            while (__any(c.x != 0)) {
                const uint2 nx2 = sh.q[k][lane];
                if (c.x != 0 && cnt < cap)
                    *reinterpret_cast<int32_t*>(rowb + ((uint32_t)cnt << 8)) = (int)c.y + __ffs(c.x) - 1;
                cnt += c.x != 0 ? 1 : 0;
                c.x &= c.x - 1;
                const bool done = c.x == 0;
                c.x = done ? nx2.x : c.x;
                c.y = done ? nx2.y : c.y;
                k = min(k + (done ? 1 : 0), qn);
            }
            __builtin_amdgcn_wave_barrier();
            qn = 0;
        };
        // candidate stream: up to 64 candidates of up to three ranges
        int jc = 0, je = 0, sg = 0;
        auto next_range = [&]() __attribute__((always_inline)) {
            jc = je = 0;
            if (pm) {
                const int v = __ffsll((unsigned long long)pm) - 1;
                pm &= pm - 1;
                jc = __builtin_amdgcn_readlane(pa, v);
                je = __builtin_amdgcn_readlane(pe, v);
                if (LE) sg = __builtin_amdgcn_readlane(psg, v);
            }
        };
        // parts 0, 1, 2: end among the chunk's candidates (e), sorted index
        // minus position (j), sheared image (s)
        struct Chunk {
            int e0, e1, e2, j0, j1, j2, s0, s1, s2;
        };
        auto part = [&](int& pos, int& e, int& j, int& s) __attribute__((always_inline)) {
            const int m = min(64 - pos, je - jc);
            j = jc - pos;
            s = sg;
            pos += m;
            e = pos;
            jc += m;
            if (jc == je) next_range();
        };
        auto take = [&]() __attribute__((always_inline)) {
            Chunk c;
            int pos = 0;
            part(pos, c.e0, c.j0, c.s0);
            part(pos, c.e1, c.j1, c.s1);
            part(pos, c.e2, c.j2, c.s2);
            return c;
        };
        auto load = [&](const Chunk& c) __attribute__((always_inline)) {
            const int k = min(ck, max(c.e2 - 1, 0));
            const int j = k + pick(k, c.e0, c.e1, c.j0, c.j1, c.j2);
            int4 q = *reinterpret_cast<const int4*>(xqb + ((uint32_t)j << 4));
            if (LE) {
                const int sj = pick(k, c.e0, c.e1, c.s0, c.s1, c.s2);
                q.x = (int)((uint32_t)q.x - (uint32_t)(sj * (int64_t)le.qd));
            }
            return q;
        };
        next_range();
        Chunk c = take();
        int4 rec = load(c);
        while (c.e2 > 0) {
            const Chunk cn = take();
            const int4 recn = load(cn);
            float fx = qdiff((uint32_t)rec.x, ox, l0), fy = qdiff((uint32_t)rec.y, oy, l1),
                  fz = qdiff((uint32_t)rec.z, oz, l2);
            float nj = fx * fx + fy * fy + fz * fz;
            // the operands of candidates 0..31 (fx, fz) and 32..63 (fy, nj)
            half_swap(fx, fy);
            half_swap(fz, nj);
#pragma unroll 1
            for (int h0 = 0; h0 < c.e2; h0 += 32) {
                f32x16 D0 = __builtin_amdgcn_mfma_f32_32x32x2f32(fx, bx0, C0, 0, 0, 0);
                f32x16 D1 = __builtin_amdgcn_mfma_f32_32x32x2f32(fx, bx1, C1, 0, 0, 0);
                D0 = __builtin_amdgcn_mfma_f32_32x32x2f32(fz, bz0, D0, 0, 0, 0);
                D1 = __builtin_amdgcn_mfma_f32_32x32x2f32(fz, bz1, D1, 0, 0, 0);
                fx = fy;
                fz = nj;
                uint32_t m = sign_bits(D0), mh = sign_bits(D1);
                half_swap(m, mh);
                m |= mh << 16;
                float near = 3.0e38f;
#pragma unroll
                for (int e = 0; e < 16; e += 2) {
                    near = fminf(fminf(fabsf(D0[e]), fabsf(D0[e + 1])), near);
                    near = fminf(fminf(fabsf(D1[e]), fabsf(D1[e + 1])), near);
                }
                if (__builtin_expect(__any(near <= delta), 0)) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        D0[e] = fabsf(D0[e]) <= delta ? -1.f : 1.f;
                        D1[e] = fabsf(D1[e]) <= delta ? -1.f : 1.f;
                    }
                    uint32_t bd = sign_bits(D0), bh = sign_bits(D1);
                    half_swap(bd, bh);
                    bd |= bh << 16;
                    const int nval = c.e2 - h0;
                    if (nval < 32) bd &= (1u << nval) - 1u;
                    if (!mine) bd = 0;
                    if (bd) {
                        const double4 xi = x[self];
                        while (bd) {
                            const int bit = __ffs(bd) - 1, k = bit + h0;
                            bd &= bd - 1;
                            const double4 xj = x[k + pick(k, c.e0, c.e1, c.j0, c.j1, c.j2)];
                            const bool in = (LE ? exact_r2_le(g, xi, xj, le.dw) : exact_r2(g, xi, xj)) < g.rv2;
                            m = (m & ~(1u << bit)) | ((in ? 1u : 0u) << bit);
                        }
                    }
                }
                if (!mine) m = 0;
                // the hits of each range, without the particle itself
                int from = 0, to = c.e0, j = c.j0;
#pragma unroll 1
                for (int q = 0; q < 3; ++q) {
                    const int b0 = max(from - h0, 0), b1 = min(to - h0, 32);
                    if (b1 > b0) {
                        const int jb = j + h0;
                        uint32_t mq = m & ((0xffffffffu >> (32 - (b1 - b0))) << b0);
                        if (jb + b0 < (int)p0 + kTile && jb + b1 > (int)p0) {
                            const uint32_t sb = (uint32_t)(self - jb);
                            if (sb < 32u) mq &= ~(1u << sb);
                        }
                        sh.q[qn][lane] = make_uint2(mq, (uint32_t)jb);
                        qn += mq ? 1 : 0;
                        if (__any(qn == kNlWords)) emit();
                    }
                    from = to;
                    to = pick(q, 1, 2, c.e1, c.e2, c.e2);
                    j = pick(q, 1, 2, c.j1, c.j2, c.j2);
                }
            }
            c = cn;
            rec = recn;
        }
        emit();
        lo = hi;
    }
    if (valid) {
        b.ncount[self] = cnt;
        if (cnt > local_max) local_max = cnt;
        if (cnt > cap) overflow = true;
        // padding to a multiple of 8 with the particle itself (as nl_one)
        for (int k = cnt; k < ((cnt + 7) & ~7) && k < cap; ++k)
            *reinterpret_cast<int32_t*>(rowb + ((uint32_t)k << 8)) = self;
        if (bonded) remap_bonded(b, n, self);
    }
}

// One wavefront per block and a few tiles in turn for each: the tiles' times
// differ by what their segments are, and wavefronts that share a block would
// hold its LDS until the last is done.
constexpr int kNlGrid = 8192;
template <bool LE>
__global__ void __launch_bounds__(kTile) k_nl_mtile(Geom g, Bufs b, int parity, int bonded) {
    __shared__ NlWave sh;
    if (!rebuild_requested(b, parity)) return;
    LeNl le{0.0, 0.0, 0u};
    if (LE) {
        le.delta = le_delta(g, b.ctl->step);
        le.dw = le_fold(g, le.delta);
        le.qd = quantize(le.delta, g.qs[0]);
    }
    int local_max = 0;
    bool overflow = false;
    const int64_t nt = (g.n + kTile - 1) / kTile, blk = xcd_block(blockIdx.x, gridDim.x);
    for (int64_t t = blk * nt / gridDim.x; t < (blk + 1) * nt / gridDim.x; ++t)
        nl_mtile<LE>(g, b, t, parity, bonded, sh, le, local_max, overflow);
    nl_epilogue(b, local_max, overflow);
}

__global__ void k_clear_rebuild(Bufs b) {
    if (threadIdx.x == 0 && blockIdx.x == 0) b.ctl->rebuild[0] = b.ctl->rebuild[1] = 0;
}

// ------------------------------------------------------------------ bonded forces

// Coordinate differences b - a for the two position formats.
struct DiffQ {
    float l0, l1, l2;
    __device__ void operator()(const int4& a, const int4& b, float& dx, float& dy, float& dz) const {
        dx = qdiff(b.x, a.x, l0);
        dy = qdiff(b.y, a.y, l1);
        dz = qdiff(b.z, a.z, l2);
    }
};
struct Diff64 {
    double L0, L1, L2, i0, i1, i2;
    __device__ void operator()(const double4& a, const double4& b, double& dx, double& dy, double& dz) const {
        dx = mimg(b.x - a.x, L0, i0);
        dy = mimg(b.y - a.y, L1, i1);
        dz = mimg(b.z - a.z, L2, i2);
    }
};

__device__ __forceinline__ void add_tensor(double* acc, double s, double rx, double ry, double rz, double fx,
                                           double fy, double fz) {
    acc[A_TXX] += s * rx * fx;
    acc[A_TYY] += s * ry * fy;
    acc[A_TZZ] += s * rz * fz;
    acc[A_TXY] += s * 0.5 * (rx * fy + ry * fx);
    acc[A_TXZ] += s * 0.5 * (rx * fz + rz * fx);
    acc[A_TYZ] += s * 0.5 * (ry * fz + rz * fy);
}

// FENE bonds and cosine bending angles acting on particle i, from its own
// rows of the sorted-space topology.  Each bond is evaluated by both ends
// (half the energy each), each angle by its three members (energy counted
// by the centre); no atomics.
// EXT (the generic FP32 kernel): the angle kinds MD_ANGLE_COSINE_SQUARED
// and MD_ANGLE_TABULATED besides the cosine bending, through
// dU/dcos(theta), theta = pi - phi the angle between b1 and b2.
template <typename Real, typename P, typename Diff, bool EXT = false>
__device__ __forceinline__ void bonded_forces(const Bufs& b, const Dyn& dyn, int64_t n, int64_t i,
                                              const P* __restrict__ xs, const P& pi, const Diff& diff,
                                              Real& fx, Real& fy, Real& fz, double* acc, bool tensor,
                                              bool& flag_bond) {
    const bool f64 = sizeof(Real) == 8;
    const int tc = b.tcnt_s[i];
    const int nb = tc & 0xff, na = tc >> 8;
    const Real K = f64 ? (Real)dyn.fene_K : (Real)dyn.fene_Kf;
    const Real R02 = f64 ? (Real)dyn.fene_R02 : (Real)dyn.fene_R02f;
    const Real hKR02 = f64 ? (Real)dyn.fene_halfKR02 : (Real)dyn.fene_halfKR02f;
    // The first kPreB bonds and kPreA angles (all of a linear chain's) load
    // their partner indices together and then gather the partners' records
    // together: two memory round trips instead of two per term.  Rows past a
    // particle's own counts hold no partner, so those gathers read the
    // particle itself and their terms are skipped; the terms are summed in
    // the same order as before.
    constexpr int kPreB = 2, kPreA = 3;
    int mb[kPreB];
    int2 ex[kPreA];
#pragma unroll
    for (int q = 0; q < kPreB; ++q) mb[q] = q < b.maxb ? b.bp_s[(int64_t)q * n + i] : 0;
#pragma unroll
    for (int q = 0; q < kPreA; ++q) ex[q] = q < b.maxa ? b.ang_s[(int64_t)q * n + i] : make_int2(0, 0);
    P pbq[kPreB], pa1[kPreA], pa2[kPreA];
#pragma unroll
    for (int q = 0; q < kPreB; ++q) pbq[q] = xs[q < nb ? mb[q] : (int)i];
#pragma unroll
    for (int q = 0; q < kPreA; ++q) {
        pa1[q] = xs[q < na ? (ex[q].x & 0x3fffffff) : (int)i];
        pa2[q] = xs[q < na ? ex[q].y : (int)i];
    }
    Real eb = 0, wb = 0;
    auto bond = [&](const P& pm) {
        Real dx, dy, dz;
        diff(pi, pm, dx, dy, dz);                    // x_m - x_i
        const Real rx = -dx, ry = -dy, rz = -dz;     // r_i - r_m
        const Real r2 = rx * rx + ry * ry + rz * rz;
        const Real qq = r2 / R02;
        if (!(qq < Real(1))) {
            flag_bond = true;
            return;
        }
        const Real om = Real(1) - qq;
        const Real fr = -K / om;
        fx += fr * rx;
        fy += fr * ry;
        fz += fr * rz;
        eb += -hKR02 * logr<Real>(om);
        wb += fr * r2;
        if (tensor) add_tensor(acc, 0.5, rx, ry, rz, fr * rx, fr * ry, fr * rz);
    };
#pragma unroll
    for (int q = 0; q < kPreB; ++q)
        if (q < nb) bond(pbq[q]);
    for (int q = kPreB; q < nb; ++q) bond(xs[b.bp_s[(int64_t)q * n + i]]);
    acc[A_EBOND] += 0.5 * (double)eb;
    acc[A_VIR] += 0.5 * (double)wb;
    const Real kb = f64 ? (Real)dyn.k_bend : (Real)dyn.k_bendf;
    Real ea = 0, wa = 0;
    auto angle = [&](const int2 e, const P& p1, const P& p2) {
        const int role = (int)((uint32_t)e.x >> 30);
        // members (A, B, C), B the centre; i is the one named by role
        const P& pa = role == 0 ? pi : p1;
        const P& pb = role == 1 ? pi : (role == 0 ? p1 : p2);
        const P& pc = role == 2 ? pi : p2;
        Real b1x, b1y, b1z, b2x, b2y, b2z;
        diff(pa, pb, b1x, b1y, b1z);                 // b1 = x_B - x_A
        diff(pb, pc, b2x, b2y, b2z);                 // b2 = x_C - x_B
        const Real l1sq = b1x * b1x + b1y * b1y + b1z * b1z;
        const Real l2sq = b2x * b2x + b2y * b2y + b2z * b2z;
        const Real il1l2 = rsq<Real>(l1sq * l2sq);
        const Real cs = (b1x * b2x + b1y * b2y + b1z * b2z) * il1l2;
        const Real i1 = rcp<Real>(l1sq), i2 = rcp<Real>(l2sq);
        Real Fx, Fy, Fz;
        if (EXT && dyn.angle_kind != MD_ANGLE_COSINE) {
            // dUdc = dU/dcos(theta); cos(phi) = -cs
            Real dUdc, ua;
            if (dyn.angle_kind == MD_ANGLE_COSINE_SQUARED) {
                const Real d = -cs - (Real)dyn.cos_phi0;
                ua = (Real)dyn.angle_K * d * d;
                dUdc = Real(-2) * (Real)dyn.angle_K * d;
            } else {
                const float cphi = (float)(-cs > Real(1) ? Real(1) : (-cs < Real(-1) ? Real(-1) : -cs));
                const float phi = acosf(cphi);
                const float q = phi * dyn.ang_idphi;
                int k = (int)q;
                k = k > dyn.ang_n - 2 ? dyn.ang_n - 2 : k;
                const float al = q - (float)k;
                const float2 t0 = dyn.ang_tab[k], t1 = dyn.ang_tab[k + 1];
                ua = (Real)((1.f - al) * t0.x + al * t1.x);
                const float gphi = (1.f - al) * t0.y + al * t1.y;       // du/dphi
                const float sn = sinf(phi);
                dUdc = (Real)(gphi / (sn > 1e-8f ? sn : 1e-8f));        // dU/dcos(theta) = -dU/dcos(phi)
            }
            const Real dA0 = b2x * il1l2 - cs * b1x * i1, dA1 = b2y * il1l2 - cs * b1y * i1,
                       dA2 = b2z * il1l2 - cs * b1z * i1;          // dcos/db1
            const Real dC0 = b1x * il1l2 - cs * b2x * i2, dC1 = b1y * il1l2 - cs * b2y * i2,
                       dC2 = b1z * il1l2 - cs * b2z * i2;          // dcos/db2
            if (role == 0) {
                Fx = dUdc * dA0; Fy = dUdc * dA1; Fz = dUdc * dA2;
                wa += -(b1x * Fx + b1y * Fy + b1z * Fz);
                if (tensor) add_tensor(acc, 1.0, -b1x, -b1y, -b1z, Fx, Fy, Fz);
            } else if (role == 2) {
                Fx = -dUdc * dC0; Fy = -dUdc * dC1; Fz = -dUdc * dC2;
                wa += b2x * Fx + b2y * Fy + b2z * Fz;
                if (tensor) add_tensor(acc, 1.0, b2x, b2y, b2z, Fx, Fy, Fz);
            } else {
                Fx = -(dUdc * dA0 - dUdc * dC0);
                Fy = -(dUdc * dA1 - dUdc * dC1);
                Fz = -(dUdc * dA2 - dUdc * dC2);
                ea += ua;
            }
        } else if (role == 0) {          // F_A = -k dcos/db1
            Fx = -kb * (b2x * il1l2 - cs * b1x * i1);
            Fy = -kb * (b2y * il1l2 - cs * b1y * i1);
            Fz = -kb * (b2z * il1l2 - cs * b1z * i1);
            wa += -(b1x * Fx + b1y * Fy + b1z * Fz);                 // (x_A - x_B) . F_A
            if (tensor) add_tensor(acc, 1.0, -b1x, -b1y, -b1z, Fx, Fy, Fz);
        } else if (role == 2) {   // F_C = k dcos/db2
            Fx = kb * (b1x * il1l2 - cs * b2x * i2);
            Fy = kb * (b1y * il1l2 - cs * b2y * i2);
            Fz = kb * (b1z * il1l2 - cs * b2z * i2);
            wa += b2x * Fx + b2y * Fy + b2z * Fz;                    // (x_C - x_B) . F_C
            if (tensor) add_tensor(acc, 1.0, b2x, b2y, b2z, Fx, Fy, Fz);
        } else {                  // F_B = -(F_A + F_C)
            Fx = kb * ((b2x * il1l2 - cs * b1x * i1) - (b1x * il1l2 - cs * b2x * i2));
            Fy = kb * ((b2y * il1l2 - cs * b1y * i1) - (b1y * il1l2 - cs * b2y * i2));
            Fz = kb * ((b2z * il1l2 - cs * b1z * i1) - (b1z * il1l2 - cs * b2z * i2));
            ea += kb * (Real(1) - cs);
        }
        fx += Fx;
        fy += Fy;
        fz += Fz;
    };
#pragma unroll
    for (int q = 0; q < kPreA; ++q)
        if (q < na) angle(ex[q], pa1[q], pa2[q]);
    for (int q = kPreA; q < na; ++q) {
        const int2 e = b.ang_s[(int64_t)q * n + i];
        angle(e, xs[e.x & 0x3fffffff], xs[e.y]);
    }
    acc[A_EANGLE] += (double)ea;
    acc[A_VIR] += (double)wa;
}

// ------------------------------------------------------------------ integration

// Velocity Verlet with the Langevin force for one particle (MODE_STEP), or
// only the on-step kinetic energy (MODE_OBSERVE / MODE_FORCES):
//   F_tot   = F(x_n) [- gamma m v' + sqrt(2 gamma m kT/dt) xi_n]
//   v_n     = v' + dt/(2m) F_tot          (v_n = v' before the first step)
//   v_{n+h} = v_n + dt/(2m) F_tot,  x_{n+1} = x_n + dt v_{n+h}, wrapped
// plus the half-skin displacement test against the build positions.
// Lees-Edwards data of one step: the offset at the new positions' step and
// the offset's change since the list was built (the rebuild criterion).
struct LeStep {
    double delta_next;     // delta(step + 1) in [0, Lx)
    double drift;          // |shear_rate Ly (step + 1 - build_step) dt|
};

__device__ __forceinline__ void finish_particle(const StepArgs& a, int64_t i, const double4& xi, int tm,
                                               const double F[3], double* acc, bool& flag_reb,
                                               bool& flag_nf, const LeStep* le = nullptr) {
    const Geom& g = a.g;
    const Bufs& b = a.b;
    const int64_t n = g.n;
    const double hdtm = a.dy.hdtm[tm];
    const double m = a.dy.mass[tm];
    double vp[3], ft[3], xbv[3];
    for (int d = 0; d < 3; ++d) vp[d] = b.v[d * n + i];
    // the build positions load with the velocities: read after the velocity
    // stores below, each would wait on its own round trip (the compiler cannot
    // move a load above a store it may alias)
    if (a.mode == MODE_STEP)
        for (int d = 0; d < 3; ++d) xbv[d] = b.xb[d * n + i];
    int32_t tg = -1;
    if (a.dy.langevin || a.mode == MODE_FORCES) tg = b.tag[i];
    if (a.dy.langevin) {
        double g0, g1, g2;
        gauss3(a.dy.seed, 0, (uint64_t)b.ctl->step, (uint64_t)tg, g0, g1, g2);
        const double gm = a.dy.gm[tm], amp = a.dy.amp[tm];
        ft[0] = (F[0] - gm * vp[0]) + amp * g0;
        ft[1] = (F[1] - gm * vp[1]) + amp * g1;
        ft[2] = (F[2] - gm * vp[2]) + amp * g2;
    } else {
        ft[0] = F[0];
        ft[1] = F[1];
        ft[2] = F[2];
    }
    const bool vh_in = b.ctl->vel_half != 0;
    double von[3], ke = 0.0;
    for (int d = 0; d < 3; ++d) {
        von[d] = vh_in ? vp[d] + hdtm * ft[d] : vp[d];
        ke += von[d] * von[d];
    }
    acc[A_EKIN] += 0.5 * m * ke;
    if (a.mode == MODE_STEP && le) {
        // sheared boundaries: crossing y = Ly (y = 0) shifts x by -delta (+delta)
        // and v_x by -shear_rate Ly (+), before the x fold; the build position
        // moves with the particle, so the displacement stays the physical one
        double xn[3], vh[3];
        for (int d = 0; d < 3; ++d) {
            vh[d] = von[d] + hdtm * ft[d];
            xn[d] = (d == 0 ? xi.x : d == 1 ? xi.y : xi.z) + a.dy.dt * vh[d];
        }
        int sc = 0;
        if (xn[1] >= g.L[1]) { xn[1] -= g.L[1]; xn[0] -= le->delta_next; vh[0] -= g.le_rate_Ly; sc = 1; }
        else if (xn[1] < 0.0) { xn[1] += g.L[1]; xn[0] += le->delta_next; vh[0] += g.le_rate_Ly; sc = -1; }
        if (sc != 0) {
            b.img[n + i] += sc;
            xbv[0] -= sc * le->delta_next;
            b.xb[i] = xbv[0];
        }
        double d2 = 0.0;
        for (int d = 0; d < 3; ++d) {
            if (xn[d] < 0.0 || xn[d] >= g.L[d]) {
                int im = b.img[d * n + i];
                if (xn[d] < 0.0) { xn[d] += g.L[d]; im -= 1; }
                if (xn[d] >= g.L[d]) { xn[d] -= g.L[d]; im += 1; }
                b.img[d * n + i] = im;
            }
            if (!isfinite(xn[d]) || !isfinite(vh[d])) flag_nf = true;
            b.v[d * n + i] = vh[d];
            const double dd = mimg(xn[d] - xbv[d], g.L[d], g.invL[d]);
            d2 += dd * dd;
        }
        // a pair's separation changes by at most both displacements plus the
        // offset's change since the build: rebuild before that reaches the skin
        if (2.0 * sqrt(d2) + le->drift >= g.skin) flag_reb = true;
        b.x[a.parity ^ 1][i] = make_double4(xn[0], xn[1], xn[2], xi.w);
        const int4 qn = quantize4(g, xn[0], xn[1], xn[2], xi.w);
        b.xq[a.parity ^ 1][i] = qn;
        if (g.x3_on) store_q3(b.x3[a.parity ^ 1], i, qn);
    } else if (a.mode == MODE_STEP) {
        double xo[3] = {xi.x, xi.y, xi.z};
        double d2 = 0.0;
        for (int d = 0; d < 3; ++d) {
            const double vh = von[d] + hdtm * ft[d];
            double xn = xo[d] + a.dy.dt * vh;
            if (xn < 0.0 || xn >= g.L[d]) {
                int im = b.img[d * n + i];
                if (xn < 0.0) { xn += g.L[d]; im -= 1; }
                if (xn >= g.L[d]) { xn -= g.L[d]; im += 1; }
                b.img[d * n + i] = im;
            }
            if (!isfinite(xn) || !isfinite(vh)) flag_nf = true;
            xo[d] = xn;
            b.v[d * n + i] = vh;
            const double dd = mimg(xn - xbv[d], g.L[d], g.invL[d]);
            d2 += dd * dd;
        }
        if (d2 > g.disp2) flag_reb = true;
        b.x[a.parity ^ 1][i] = make_double4(xo[0], xo[1], xo[2], xi.w);
        const int4 qn = quantize4(g, xo[0], xo[1], xo[2], xi.w);
        b.xq[a.parity ^ 1][i] = qn;
        if (g.x3_on) store_q3(b.x3[a.parity ^ 1], i, qn);
    } else if (a.mode == MODE_FORCES && a.f_out) {
        a.f_out[3 * (int64_t)tg] = F[0];
        a.f_out[3 * (int64_t)tg + 1] = F[1];
        a.f_out[3 * (int64_t)tg + 2] = F[2];
    }
}

// First row of a step's partial sums: without the tensor the two parities'
// sums lie side by side, so that a step's are there while the next step runs.
__device__ __forceinline__ int partial_row(int nacc, int parity) { return nacc < kNacc ? parity * nacc : 0; }

// Flags (one store or atomic per wave) and the deterministic block
// reduction of the per-particle sums into partials[k][block]; BS threads per
// block.
template <int BS = kBlock>
__device__ __forceinline__ void block_epilogue(const StepArgs& a, const double* acc, bool flag_reb,
                                              bool flag_bond, bool flag_nf, int nacc, int64_t slot, int64_t nslots) {
    const Bufs& b = a.b;
    const bool any_reb = __any(flag_reb);
    const bool any_bond = __any(flag_bond);
    const bool any_nf = __any(flag_nf);
    if ((threadIdx.x & 63) == 0) {
        // Stores to one address from many wavefronts serialize, and under a
        // drifting sheared image nearly every wavefront of a step can ask for
        // the rebuild, so a wavefront sets the flag only when it reads it
        // clear; a stale read costs one redundant store, never a lost request.
        uint32_t* const next = &b.ctl->rebuild[a.parity ^ 1];
        if (any_reb && __hip_atomic_load(next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u)
            __atomic_store_n(next, 1u, __ATOMIC_RELAXED);
        if (any_bond) atomicOr(&b.ctl->status, MD_FLAG_BOND_BROKEN);
        if (any_nf) atomicOr(&b.ctl->status, MD_FLAG_NONFINITE);
    }
    __shared__ double red[BS / 64][kNacc];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int q = 0; q < nacc; ++q) {
        const double s = wave_sum(acc[q]);
        if (lane == 0) red[w][q] = s;
    }
    __syncthreads();
    if ((int)threadIdx.x < nacc) {
        double s = 0.0;
        for (int ww = 0; ww < BS / 64; ++ww) s += red[ww][threadIdx.x];
        b.partials[((int64_t)threadIdx.x + partial_row(nacc, a.parity)) * nslots + slot] = s;
    }
}

// One block of BS threads: reduce the step's partials[k][block] in a fixed
// order and record its observables.  MODE_STEP (the end of a call) also
// advances the step counter; MODE_PREV, the first block of the next step's
// kernel, finds it advanced.  NACC: the quantities the step kernel summed (the
// virial tensor only when it was asked for).
constexpr int kFinal = 1024;
constexpr int kNaccStep = A_VIR + 1;
template <int BS, int NACC>
__device__ __forceinline__ void finalize_body(const Bufs& b, int parity, int nblocks, int mode, const double* spart) {
    __shared__ double red[BS / 64][NACC];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const double* __restrict__ part = b.partials + (int64_t)partial_row(NACC, parity) * nblocks;
    double s[NACC];
#pragma unroll
    for (int k = 0; k < NACC; ++k) s[k] = 0.0;
    for (int blk0 = 0; blk0 < nblocks; blk0 += 4 * BS) {
        double v[4][NACC];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int blk = blk0 + r * BS + threadIdx.x;
#pragma unroll
            for (int k = 0; k < NACC; ++k) v[r][k] = blk < nblocks ? part[(int64_t)k * nblocks + blk] : 0.0;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int k = 0; k < NACC; ++k) s[k] += v[r][k];
        if (spart)
            for (int r = 0; r < 4; ++r) {
                const int blk = blk0 + r * BS + threadIdx.x;
                if (blk < nblocks) s[A_EPAIR] += spart[blk];
            }
    }
#pragma unroll
    for (int k = 0; k < NACC; ++k) {
        const double t = wave_sum(s[k]);
        if (lane == 0) red[w][k] = t;
    }
    __syncthreads();
    // one lane per quantity sums the wavefront totals (fixed order), so the
    // serial part below reads finished sums only
    __shared__ double fin[NACC];
    if (threadIdx.x < NACC) {
        double v = 0.0;
        for (int ww = 0; ww < BS / 64; ++ww) v += red[ww][threadIdx.x];
        fin[threadIdx.x] = v;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        DevCtl* c = b.ctl;
        const bool prev = mode == MODE_PREV;
        const int64_t step = c->step - (prev ? 1 : 0);
        double rec[kHistRec];
        rec[H_STEP] = (double)step;
        rec[H_EPAIR] = fin[A_EPAIR];
        rec[H_EBOND] = fin[A_EBOND];
        rec[H_EANGLE] = fin[A_EANGLE];
        rec[H_EKIN] = fin[A_EKIN];
        rec[H_VIR] = fin[A_VIR];
        for (int k = 0; k < 6; ++k) rec[H_T0 + k] = NACC == kNacc ? fin[(A_TXX + k) % NACC] : 0.0;
        rec[H_NREB] = (double)(prev ? c->prev_rebuilds : c->n_rebuilds);
        rec[H_STATUS] = (double)(prev ? c->prev_status : c->status);
        rec[H_NLMAX] = (double)(prev ? c->prev_nl_max : c->nl_max);
        rec[15] = 0.0;
        for (int k = 0; k < kHistRec; ++k) b.cur[k] = rec[k];
        if (prev || mode == MODE_STEP) {
            double* h = b.hist + (int64_t)(step % MD_HISTORY_CAPACITY) * kHistRec;
            for (int k = 0; k < kHistRec; ++k) h[k] = rec[k];
        }
        if (mode == MODE_STEP) {
            c->step = step + 1;
            c->vel_half = 1;
            c->ran = 0;
        }
        if (mode == MODE_OBSERVE || mode == MODE_FORCES) c->rebuild[0] = c->rebuild[1] = 0;
    }
}

template <int BS, int NACC>
__global__ void __launch_bounds__(BS) k_finalize(Bufs b, int parity, int nblocks, int mode, const double* spart) {
    finalize_body<BS, NACC>(b, parity, nblocks, mode, spart);
}

// Block index and grid of a step kernel without the block that writes the
// previous step's record (StepArgs::fin): true for that block, its work done.
// It comes first, so that its serial tail lies beside the other blocks' work.
template <int BS = kBlock>
__device__ __forceinline__ bool finalize_block(const StepArgs& a, int& blk, int& grid) {
    blk = (int)blockIdx.x - a.fin;
    grid = (int)gridDim.x - a.fin;
    if (blk >= 0) return false;
    if (a.b.ctl->fin_prev) finalize_body<BS, kNaccStep>(a.b, a.parity ^ 1, grid, MODE_PREV, a.fin_spart);
    return true;
}

// ------------------------------------------------------------------ step kernels

// FP64 pair path: FP64 positions gathered from the double-buffered double4
// array, all pair and bonded math in FP64.
template <bool SINGLE, bool BONDED, int BS>
__global__ void __launch_bounds__(BS) k_step64(const StepArgs a) {
    int blk, grid;
    if (finalize_block<BS>(a, blk, grid)) return;
    const Geom& g = a.g;
    const Bufs& b = a.b;
    const int64_t n = g.n;
    const double4* __restrict__ xin = b.x[a.parity];
    double acc[kNacc];
#pragma unroll
    for (int k = 0; k < kNacc; ++k) acc[k] = 0.0;
    bool flag_reb = false, flag_bond = false, flag_nf = false;
    const bool tensor = a.tensor != 0;
    const int64_t ntile = (n + BS - 1) / BS;
    const int64_t bt = xcd_block(blk, grid);
    for (int64_t t = bt * ntile / grid; t < (bt + 1) * ntile / grid; ++t) {
    const int64_t i = t * BS + threadIdx.x;
    if (i < n) {
        const double4 xi = xin[i];
        const int ti = SINGLE ? 0 : (int)xi.w;
        double fx = 0, fy = 0, fz = 0, ui = 0, wi = 0;
        int cnt = b.ncount[i];
        cnt = cnt < g.cap ? cnt : g.cap;
        const int32_t* __restrict__ row = b.nl + nl_base(i, g.cap);
        for (int k = 0; k < cnt; ++k) {
            const double4 xj = xin[row[nl_off(k)]];
            const double dx = mimg(xj.x - xi.x, g.L[0], g.invL[0]);
            const double dy = mimg(xj.y - xi.y, g.L[1], g.invL[1]);
            const double dz = mimg(xj.z - xi.z, g.L[2], g.invL[2]);
            const double r2 = dx * dx + dy * dy + dz * dz;
            const int tp = SINGLE ? 0 : ti * MD_MAX_TYPES + (int)xj.w;
            if (exact_r2(g, xi, xj) < a.pt.rc2d[tp]) {
                const PairCoef<double>& c = a.pt.d[tp];
                double fr, u;
                if (c.cap2 > 0.0 && r2 < c.cap2) {
                    fr = c.fcap / sqrt(r2);
                    u = c.ucap;
                } else {
                    const double inv = 1.0 / r2;
                    const double s2 = c.sig2 * inv;
                    const double s6 = s2 * s2 * s2;
                    fr = c.eps24 * s6 * (2.0 * s6 - 1.0) * inv;
                    u = c.eps4 * s6 * (s6 - 1.0) - c.shift;
                }
                fx -= fr * dx;
                fy -= fr * dy;
                fz -= fr * dz;
                ui += u;
                wi += fr * r2;
                if (tensor) add_tensor(acc, 0.5, -dx, -dy, -dz, -fr * dx, -fr * dy, -fr * dz);
            }
        }
        acc[A_EPAIR] += 0.5 * ui;
        acc[A_VIR] += 0.5 * wi;
        if (BONDED) {
            const Diff64 df{g.L[0], g.L[1], g.L[2], g.invL[0], g.invL[1], g.invL[2]};
            bonded_forces<double, double4, Diff64>(b, a.dy, n, i, xin, xi, df, fx, fy, fz, acc, tensor, flag_bond);
        }
        const double F[3] = {fx, fy, fz};
        finish_particle(a, i, xi, SINGLE ? 0 : ti, F, acc, flag_reb, flag_nf);
    }
    }
    block_epilogue<BS>(a, acc, flag_reb, flag_bond, flag_nf, tensor ? kNacc : kNaccStep, blk, grid);
}

// FP32 pair path.  Neighbours are gathered as 16-byte fixed-point records;
// dx = (int32)(q_j - q_i) * L/2^32 is the minimum image with no branch and
// an absolute error of a few 1e-8; the pair and bonded math is FP32.  A
// cutoff decision inside the rounding band around rc is retaken in FP64
// from the FP64 positions, so the set of interacting pairs is that of the
// FP64 definition.  Neighbour indices are loaded one batch of 8 ahead of
// the gathers that use them.
template <bool SINGLE, bool BONDED, bool TENSOR, int BS>
__global__ void __launch_bounds__(BS) k_step_q(const StepArgs a) {
    int blk, grid;
    if (finalize_block<BS>(a, blk, grid)) return;
    const Geom& g = a.g;
    const Bufs& b = a.b;
    const int64_t n = g.n;
    const int4* __restrict__ xq = b.xq[a.parity];
    const double4* __restrict__ x64 = b.x[a.parity];
    double acc[kNacc];
#pragma unroll
    for (int k = 0; k < kNacc; ++k) acc[k] = 0.0;
    bool flag_reb = false, flag_bond = false, flag_nf = false;
    const int64_t ntile = (n + BS - 1) / BS;
    const int64_t bt = xcd_block(blk, grid);
    for (int64_t t = bt * ntile / grid; t < (bt + 1) * ntile / grid; ++t) {
    const int64_t i = t * BS + threadIdx.x;
    if (i < n) {
        const double4 xi = x64[i];
        const int4 qi = quantize4(g, xi.x, xi.y, xi.z, xi.w);  // equals xq[i]: same function
        const int ti = SINGLE ? 0 : qi.w;
        const float l0 = g.ql[0], l1 = g.ql[1], l2 = g.ql[2];
        float fx = 0.f, fy = 0.f, fz = 0.f, ue = 0.f, we = 0.f;
        float txx = 0.f, tyy = 0.f, tzz = 0.f, txy = 0.f, txz = 0.f, tyz = 0.f;
        int cnt = b.ncount[i];
        cnt = cnt < g.cap ? cnt : g.cap;
        const int32_t* __restrict__ row = b.nl + nl_base(i, g.cap);
        const int self = (int)i;

        auto pair = [&](const int4& qj, int j, bool valid) {
            const float dx = qdiff(qj.x, qi.x, l0);
            const float dy = qdiff(qj.y, qi.y, l1);
            const float dz = qdiff(qj.z, qi.z, l2);
            const float r2 = dx * dx + dy * dy + dz * dz;
            const int tp = SINGLE ? 0 : ti * MD_MAX_TYPES + qj.w;
            bool in = valid && r2 < a.pt.rc2lo[tp];
            if (valid && !in && r2 < a.pt.rc2hi[tp]) in = exact_r2(g, xi, x64[j]) < a.pt.rc2d[tp];
            if (in) {
                const PairCoef<float>& c = a.pt.f[tp];
                float fr, u;
                if (a.pt.tabn[tp] > 1) {
                    // tabulated: u and f = -du/dr linear in r on the pair's grid
                    const float r = sqrtf(r2);
                    float q = (r - a.pt.tab_rmin[tp]) * a.pt.tab_idr[tp];
                    q = q > 0.f ? q : 0.f;
                    int kq = (int)q;
                    kq = kq > a.pt.tabn[tp] - 2 ? a.pt.tabn[tp] - 2 : kq;
                    const float al = q - (float)kq;
                    const float2* trow = b.tab + (int64_t)tp * g.table_points;
                    const float2 t0 = trow[kq], t1 = trow[kq + 1];
                    u = (1.f - al) * t0.x + al * t1.x;
                    fr = ((1.f - al) * t0.y + al * t1.y) * __builtin_amdgcn_rcpf(r);
                } else if (c.cap2 > 0.f && r2 < c.cap2) {
                    fr = c.fcap * __builtin_amdgcn_rsqf(r2);
                    u = c.ucap;
                } else {
                    const float inv = __builtin_amdgcn_rcpf(r2);
                    const float s2 = c.sig2 * inv;
                    const float s6 = s2 * s2 * s2;
                    fr = c.eps24 * s6 * (2.f * s6 - 1.f) * inv;
                    u = c.eps4 * s6 * (s6 - 1.f) - c.shift;
                }
                fx -= fr * dx;
                fy -= fr * dy;
                fz -= fr * dz;
                ue += u;
                we += fr * r2;
                if (TENSOR) {
                    txx += fr * dx * dx; tyy += fr * dy * dy; tzz += fr * dz * dz;
                    txy += fr * dx * dy; txz += fr * dx * dz; tyz += fr * dy * dz;
                }
            }
        };

        // Neighbour indices are prefetched one batch of 8 ahead.  The loads
        // are unconditional (slot clamped inside the row capacity) so the
        // compiler can count them and wait only for the gathers in use;
        // slots past the row's count select the particle itself, masked.
        constexpr int B = 8;
        const int last = cnt > 0 ? cnt - 1 : 0;   // loads past the row repeat its last slot
        const char* __restrict__ xqb = reinterpret_cast<const char*>(xq);
        int jn[B];
#pragma unroll
        for (int u = 0; u < B; ++u) {
            const int v = row[nl_off(u < last ? u : last)];
            jn[u] = u < cnt ? v : self;
        }
        for (int k0 = 0; k0 < cnt; k0 += B) {
            int jc[B];
            int4 q[B];
#pragma unroll
            for (int u = 0; u < B; ++u) {
                jc[u] = jn[u];
                q[u] = *reinterpret_cast<const int4*>(xqb + ((uint32_t)jc[u] << 4));
            }
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const int kk = k0 + B + u;
                const int v = row[nl_off(kk < last ? kk : last)];
                jn[u] = kk < cnt ? v : self;
            }
#pragma unroll
            for (int u = 0; u < B; ++u) pair(q[u], jc[u], k0 + u < cnt);
        }
        acc[A_EPAIR] += 0.5 * (double)ue;
        acc[A_VIR] += 0.5 * (double)we;
        if (TENSOR) {
            acc[A_TXX] += 0.5 * (double)txx; acc[A_TYY] += 0.5 * (double)tyy; acc[A_TZZ] += 0.5 * (double)tzz;
            acc[A_TXY] += 0.5 * (double)txy; acc[A_TXZ] += 0.5 * (double)txz; acc[A_TYZ] += 0.5 * (double)tyz;
        }
        if (BONDED) {
            const DiffQ df{l0, l1, l2};
            bonded_forces<float, int4, DiffQ>(b, a.dy, n, i, xq, qi, df, fx, fy, fz, acc, TENSOR, flag_bond);
        }
        const double F[3] = {(double)fx, (double)fy, (double)fz};
        finish_particle(a, i, xi, SINGLE ? 0 : ti, F, acc, flag_reb, flag_nf);
    }
    }
    block_epilogue<BS>(a, acc, flag_reb, flag_bond, flag_nf, TENSOR ? kNacc : kNaccStep, blk, grid);
}


// FP32 fast path: one particle type, cubic box, no capping radius.  The pair
// math runs in fixed-point length units (u = L / 2^32): r2 = |dq|^2, the
// coefficients are rescaled on the host, out-of-range pairs get inv = 0 so
// that every term vanishes without a branch, and the FP64 re-decision of the
// rounding band around rc costs one rarely taken branch per batch of 8.
//   F_i = -(24 eps / u) sum a b-weighted dq,  a = s6 (2 s6 - 1), b = a / r2
//   U_i = 1/2 (4 eps sum s6 (s6 - 1) - n_in shift),  W_i = 1/2 24 eps sum a
template <bool BONDED, bool TENSOR>
__device__ __forceinline__ void fast_particle(const StepArgs& a, int64_t i, double* acc, bool& flag_reb,
                                              bool& flag_bond, bool& flag_nf) {
    const Geom& g = a.g;
    const Bufs& b = a.b;
    const int64_t n = g.n;
    const int4* __restrict__ xq = b.xq[a.parity];
    const double4* __restrict__ x64 = b.x[a.parity];
    {
        const double4 xi = x64[i];
        const int4 qi = quantize4(g, xi.x, xi.y, xi.z, xi.w);  // equals xq[i]: same function
        const FastCoef& fc = a.fast;
        float fx = 0.f, fy = 0.f, fz = 0.f, ea = 0.f, wa = 0.f, nin = 0.f;
        float txx = 0.f, tyy = 0.f, tzz = 0.f, txy = 0.f, txz = 0.f, tyz = 0.f;
        int cnt = b.ncount[i];
        cnt = cnt < g.cap ? cnt : g.cap;
        // the capacity is a multiple of 8, so the padded row stays inside it
        const int nslots = min((cnt + 7) & ~7, g.cap);
        const int32_t* __restrict__ row = b.nl + nl_base(i, g.cap);
        // unbonded: 12-byte records (Geom::x3_on); bonded: the 16-byte ones
        const char* __restrict__ recb = BONDED ? reinterpret_cast<const char*>(xq)
                                              : reinterpret_cast<const char*>(b.x3[a.parity]);
        const int last = nslots > 0 ? nslots - 1 : 0;  // loads past the row repeat its last slot
        // Indices are loaded two batches ahead of their gathers (16 loads
        // of 256 bytes in flight per wavefront) to cover HBM latency.
        constexpr int B = 8;
        int jn[B], jn2[B];
#pragma unroll
        for (int u = 0; u < B; ++u) {
            jn[u] = row[(u < last ? u : last) * kTile];
            jn2[u] = row[(B + u < last ? B + u : last) * kTile];
        }
        for (int k0 = 0; k0 < nslots; k0 += B) {
            int jc[B];
            Q3 q[B];
#pragma unroll
            for (int u = 0; u < B; ++u) {
                jc[u] = jn[u];
                if (BONDED) {
                    const int4 r = *reinterpret_cast<const int4*>(recb + ((uint32_t)jc[u] << 4));
                    q[u] = Q3{r.x, r.y, r.z};
                } else {
                    q[u] = *reinterpret_cast<const Q3*>(recb + (uint32_t)jc[u] * 12u);
                }
            }
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const int kk = k0 + 2 * B + u;
                jn[u] = jn2[u];
                jn2[u] = row[nl_off(kk < last ? kk : last)];
            }
            float dx[B], dy[B], dz[B], r2[B];
            uint32_t inmask = 0, bandmask = 0;
#pragma unroll
            for (int u = 0; u < B; ++u) {
                dx[u] = (float)(int32_t)((uint32_t)q[u].x - (uint32_t)qi.x);
                dy[u] = (float)(int32_t)((uint32_t)q[u].y - (uint32_t)qi.y);
                dz[u] = (float)(int32_t)((uint32_t)q[u].z - (uint32_t)qi.z);
                r2[u] = dx[u] * dx[u] + dy[u] * dy[u] + dz[u] * dz[u];
                // r2 > 0 excludes the padding self entries
                const bool lo = r2[u] > 0.f && r2[u] < fc.rc2lo;
                const bool band = r2[u] >= fc.rc2lo && r2[u] < fc.rc2hi;
                inmask |= (uint32_t)lo << u;
                bandmask |= (uint32_t)band << u;
            }
            if (__builtin_expect(bandmask != 0, 0)) {
#pragma unroll
                for (int u = 0; u < B; ++u)
                    if ((bandmask >> u) & 1u)
                        if (exact_r2(g, xi, x64[jc[u]]) < fc.rc2d) inmask |= 1u << u;
            }
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const bool in = (inmask >> u) & 1u;
                const float inv = in ? __builtin_amdgcn_rcpf(r2[u]) : 0.f;
                const float s2 = fc.sig2u * inv;
                const float s6 = s2 * s2 * s2;
                const float aa = s6 * (2.f * s6 - 1.f);
                const float bb = aa * inv;
                fx += bb * dx[u];
                fy += bb * dy[u];
                fz += bb * dz[u];
                wa += aa;
                ea += s6 * s6 - s6;
                nin += in ? 1.f : 0.f;
                if (TENSOR) {
                    txx += bb * dx[u] * dx[u]; tyy += bb * dy[u] * dy[u]; tzz += bb * dz[u] * dz[u];
                    txy += bb * dx[u] * dy[u]; txz += bb * dx[u] * dz[u]; tyz += bb * dy[u] * dz[u];
                }
            }
        }
        fx *= -fc.eps24_u;
        fy *= -fc.eps24_u;
        fz *= -fc.eps24_u;
        acc[A_EPAIR] += 0.5 * ((double)fc.eps4 * (double)ea - (double)fc.shift * (double)nin);
        acc[A_VIR] += 0.5 * (double)fc.eps24 * (double)wa;
        if (TENSOR) {
            // r_ij f_ij = 24 eps b dq dq (units cancel: b carries 1/u^2)
            const double s = 0.5 * (double)fc.eps24;
            acc[A_TXX] += s * txx; acc[A_TYY] += s * tyy; acc[A_TZZ] += s * tzz;
            acc[A_TXY] += s * txy; acc[A_TXZ] += s * txz; acc[A_TYZ] += s * tyz;
        }
        if (BONDED) {
            const DiffQ df{g.ql[0], g.ql[1], g.ql[2]};
            bonded_forces<float, int4, DiffQ>(b, a.dy, n, i, xq, qi, df, fx, fy, fz, acc, TENSOR, flag_bond);
        }
        const double F[3] = {(double)fx, (double)fy, (double)fz};
        finish_particle(a, i, xi, 0, F, acc, flag_reb, flag_nf);
    }
}

// BS particles per block (64 .. 512, the block dimension the autotuner
// picks); one block per BS-particle tile, blocks in XCD-contiguous order.
template <bool BONDED, bool TENSOR, int BS>
__device__ __forceinline__ void step_fast_body(const StepArgs& a) {
    int blk, grid;
    if (finalize_block<BS>(a, blk, grid)) return;
    const int64_t n = a.g.n;
    double acc[kNacc];
#pragma unroll
    for (int k = 0; k < kNacc; ++k) acc[k] = 0.0;
    bool flag_reb = false, flag_bond = false, flag_nf = false;
    const int64_t ntile = (n + BS - 1) / BS;
    const int64_t bt = xcd_block(blk, grid);
    for (int64_t t = bt * ntile / grid; t < (bt + 1) * ntile / grid; ++t) {
        const int64_t i = t * BS + threadIdx.x;
        if (i < n) fast_particle<BONDED, TENSOR>(a, i, acc, flag_reb, flag_bond, flag_nf);
    }
    block_epilogue<BS>(a, acc, flag_reb, flag_bond, flag_nf, TENSOR ? kNacc : kNaccStep, blk, grid);
}

// The LJ form: 139-142 VGPRs, 3 wavefronts per SIMD, at every block size.
template <bool TENSOR, int BS>
__global__ void __launch_bounds__(BS)
k_step_fast(const StepArgs a) {
    step_fast_body<false, TENSOR, BS>(a);
}

// The bonded form is capped at 128 VGPRs (4 wavefronts per SIMD instead of
// 3, a few bytes of spill): 6% faster on the 2M-bead melt, whose list is
// short and whose bonded partners add gathers; the same cap costs the LJ
// kernel 4%, so it keeps its 144 registers.
template <bool TENSOR, int BS>
__global__ void __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(4)))
k_step_fast_bonded(const StepArgs a) {
    step_fast_body<true, TENSOR, BS>(a);
}

// AdResS weight of a position x along the slab axis: 1 within d_at of x0
// (minimum image), cos^2(pi (d - d_at) / (2 d_hy)) over the hybrid zone, 0
// beyond.
__device__ __forceinline__ float adress_weight(const Dyn& dy, float x, float Lx) {
    float d = x - dy.ad_x0;
    if (d > 0.5f * Lx) d -= Lx;
    else if (d < -0.5f * Lx) d += Lx;
    d = fabsf(d);
    if (d < dy.ad_dat) return 1.f;
    if (d >= dy.ad_dat + dy.ad_dhy) return 0.f;
    // cos^2 z = (1 + cos 2z) / 2, with the revolution-scaled hardware cosine
    return 0.5f + 0.5f * __builtin_amdgcn_cosf(dy.ad_k * (d - dy.ad_dat) * 0.3183098861837907f);
}

// theta_ij of the DPD thermostat: Philox4x32-10 at counter (step low word,
// step high word, min id, max id) with key (seed low word, seed high word
// ^ 6), Box-Muller on the first two words as uniforms (w + 1/2) 2^-32,
// evaluated in FP32 with the hardware log2 and cosine (cos(2 pi u) from the
// revolution-scaled instruction): within a few 1e-7 of the FP64 draw, far
// below the FP32 force rounding.
__device__ __forceinline__ float dpd_theta(uint64_t seed, uint64_t step, uint32_t ti, uint32_t tj) {
    uint32_t x0 = (uint32_t)step, x1 = (uint32_t)(step >> 32), x2 = ti < tj ? ti : tj, x3 = ti < tj ? tj : ti;
    philox4x32_10(x0, x1, x2, x3, (uint32_t)seed, (uint32_t)(seed >> 32) ^ 6u);
    const float u0 = fmaf((float)x0, 0x1.0p-32f, 0x1.0p-33f);
    const float u1 = fmaf((float)x1, 0x1.0p-32f, 0x1.0p-33f);
    // -2 ln u0 = -2 ln 2 log2 u0
    const float rr = sqrtf(-1.3862943611198906f * __builtin_amdgcn_logf(u0));
    return rr * __builtin_amdgcn_cosf(u1);
}

// Generic FP32 step, one 256-particle tile per block, for what the fast
// kernels leave out: the DPD pair thermostat (MD_DPD), Lees-Edwards shear,
// tabulated pair potentials and the angle kinds beyond the cosine bending.
// The pair table (any types, capping radius, or a tabulated pair: u and f
// interpolated linearly in r) and the bonded terms under the sheared minimum
// image, the DPD forces from the half-step velocities (MODE_STEP only: a
// thermostat force, not part of md_forces), then the integration with the
// sheared boundary crossing.  The DPD pair force on i, with e = (r_i - r_j)/r, w = 1 - r/rc_d:
//   (-gamma w^2 (e . v_ij) + sigma w theta_ij / sqrt(dt)) e,
// computed by both members of a pair with the same theta_ij, so the two
// contributions cancel to FP32 rounding.
// SINGLE: one particle type, so the pair parameters are uniform and held in
// scalar registers.  LDSTAB: the tables the kernel reads (the pair row of
// type pair 0 and the AdResS coarse-grained row) are first copied into LDS,
// [2][table_points] (u, f) pairs, so that their lookups do not wait on
// global memory.  The neighbour row is pipelined: the index two slots ahead
// and the record (and DPD velocity) one slot ahead of the pair arithmetic.
template <bool BONDED, bool SINGLE, bool LDSTAB, int BS>
__global__ void __launch_bounds__(BS) k_step_gen(const StepArgs a) {
    extern __shared__ float2 stab[];
    int blk, grid;
    if (finalize_block<BS>(a, blk, grid)) return;
    const Geom& g = a.g;
    const Bufs& b = a.b;
    const int64_t n = g.n;
    const int4* __restrict__ xq = b.xq[a.parity];
    const double4* __restrict__ x64 = b.x[a.parity];
    if (LDSTAB) {
        const int np = g.table_points;
        const float2* __restrict__ src0 = b.tab;
        const float2* __restrict__ src1 = b.tab + (int64_t)kCgTableRow * np;
        for (int k = threadIdx.x; k < np; k += BS) {
            stab[k] = src0[k];
            stab[np + k] = src1[k];
        }
        __syncthreads();
    }
    double acc[kNacc];
#pragma unroll
    for (int k = 0; k < kNacc; ++k) acc[k] = 0.0;
    bool flag_reb = false, flag_bond = false, flag_nf = false;
    const bool tensor = a.tensor != 0;
    const int64_t step = b.ctl->step;
    double delta = 0.0, dw = 0.0;
    uint32_t qd = 0;
    LeStep les{0.0, 0.0};
    if (g.le) {
        delta = le_delta(g, step);
        dw = le_fold(g, delta);
        qd = quantize(delta, g.qs[0]);
        les.delta_next = le_delta(g, step + 1);
        les.drift = fabs(g.le_rate_Ly * ((double)(step + 1 - b.ctl->build_step) * g.le_dt));
    }
    const bool dpd = a.dy.dpd && a.mode == MODE_STEP;
    const int64_t i = (int64_t)xcd_block(blk, grid) * BS + threadIdx.x;
    if (i < n) {
        const double4 xi = x64[i];
        const int4 qi = quantize4(g, xi.x, xi.y, xi.z, xi.w);
        const int ti = qi.w;
        const DiffLEQ df{g.ql[0], g.ql[1], g.ql[2], qd};
        float fx = 0.f, fy = 0.f, fz = 0.f, ue = 0.f, we = 0.f;
        float txx = 0.f, tyy = 0.f, tzz = 0.f, txy = 0.f, txz = 0.f, tyz = 0.f;
        const float wi = a.dy.adress ? adress_weight(a.dy, (float)xi.x, (float)g.L[0]) : 1.f;
        // DPD reads the half-step velocities and ids from the snapshot in
        // b.vt taken before this kernel (b.v is overwritten here as particles
        // finish): one 16-byte record (vx, vy, vz, id) per particle
        const float4* __restrict__ vs = reinterpret_cast<const float4*>(b.vt);
        float4 vi = make_float4(0.f, 0.f, 0.f, 0.f);
        if (dpd) vi = vs[i];
        int cnt = b.ncount[i];
        cnt = cnt < g.cap ? cnt : g.cap;
        const int32_t* __restrict__ row = b.nl + nl_base(i, g.cap);
        // slots past the end repeat the last one (every slot below cnt holds
        // a particle index); an empty row reads the particle itself
        const int last = cnt > 0 ? cnt - 1 : 0;
        auto slot = [&](int k) { return cnt > 0 ? row[nl_off(k < last ? k : last)] : (int)i; };
        int jA = slot(0), jB = slot(1);
        int4 qA = xq[jA];
        float4 vA = dpd ? vs[jA] : make_float4(0.f, 0.f, 0.f, 0.f);
        for (int k = 0; k < cnt; ++k) {
            const int j = jA;
            const int4 qj = qA;
            const float4 vj = vA;
            jA = jB;
            jB = slot(k + 2);
            qA = xq[jA];
            if (dpd) vA = vs[jA];
            float dx, dy, dz;
            const int s = df(qi, qj, dx, dy, dz);
            const float r2 = dx * dx + dy * dy + dz * dz;
            const int tp = SINGLE ? 0 : ti * MD_MAX_TYPES + qj.w;
            bool in = r2 < a.pt.rc2lo[tp];
            if (!in && r2 < a.pt.rc2hi[tp]) in = exact_r2_le(g, xi, x64[j], dw) < a.pt.rc2d[tp];
            // AdResS: the coarse-grained force of the pair, to be mixed in below
            bool cg_in = false;
            float ucg = 0.f, frcg = 0.f;
            if (a.dy.adress && a.pt.cgn[tp] > 1) {
                cg_in = r2 < a.pt.cg_rc2lo[tp];
                if (!cg_in && r2 < a.pt.cg_rc2hi[tp]) cg_in = exact_r2_le(g, xi, x64[j], dw) < a.pt.cg_rc2d[tp];
                if (cg_in) {
                    const float r = sqrtf(r2);
                    float q = (r - a.pt.cg_rmin[tp]) * a.pt.cg_idr[tp];
                    q = q > 0.f ? q : 0.f;
                    int kq = (int)q;
                    kq = kq > a.pt.cgn[tp] - 2 ? a.pt.cgn[tp] - 2 : kq;
                    const float al = q - (float)kq;
                    const float2* trow = LDSTAB ? stab + g.table_points
                                                : b.tab + (int64_t)(kCgTableRow + tp) * g.table_points;
                    const float2 t0 = trow[kq], t1 = trow[kq + 1];
                    ucg = (1.f - al) * t0.x + al * t1.x;
                    frcg = ((1.f - al) * t0.y + al * t1.y) * __builtin_amdgcn_rcpf(r);
                }
            }
            if (in || cg_in) {
                const PairCoef<float>& c = a.pt.f[tp];
                float fr = 0.f, u = 0.f;
                if (!in) {
                } else if (a.pt.tabn[tp] > 1) {
                    // tabulated: u and f = -du/dr linear in r on the pair's grid
                    const float r = sqrtf(r2);
                    float q = (r - a.pt.tab_rmin[tp]) * a.pt.tab_idr[tp];
                    q = q > 0.f ? q : 0.f;
                    int kq = (int)q;
                    kq = kq > a.pt.tabn[tp] - 2 ? a.pt.tabn[tp] - 2 : kq;
                    const float al = q - (float)kq;
                    const float2* trow = LDSTAB ? stab : b.tab + (int64_t)tp * g.table_points;
                    const float2 t0 = trow[kq], t1 = trow[kq + 1];
                    u = (1.f - al) * t0.x + al * t1.x;
                    fr = ((1.f - al) * t0.y + al * t1.y) * __builtin_amdgcn_rcpf(r);
                } else if (c.cap2 > 0.f && r2 < c.cap2) {
                    fr = c.fcap * __builtin_amdgcn_rsqf(r2);
                    u = c.ucap;
                } else {
                    const float inv = __builtin_amdgcn_rcpf(r2);
                    const float s2 = c.sig2 * inv;
                    const float s6 = s2 * s2 * s2;
                    fr = c.eps24 * s6 * (2.f * s6 - 1.f) * inv;
                    u = c.eps4 * s6 * (s6 - 1.f) - c.shift;
                }
                if (a.dy.adress) {
                    // x_j from its fixed-point coordinate (positions lie in [0, L))
                    const float lam = wi * adress_weight(a.dy, (float)(uint32_t)qj.x * g.ql[0], (float)g.L[0]);
                    u = lam * u + (1.f - lam) * ucg;
                    fr = lam * fr + (1.f - lam) * frcg;
                }
                fx -= fr * dx;
                fy -= fr * dy;
                fz -= fr * dz;
                ue += u;
                we += fr * r2;
                if (tensor) {
                    txx += fr * dx * dx; tyy += fr * dy * dy; tzz += fr * dz * dz;
                    txy += fr * dx * dy; txz += fr * dx * dz; tyz += fr * dy * dz;
                }
            }
            if (dpd && r2 < a.dy.dpd_rc2 && r2 > 0.f) {
                const float ir = __builtin_amdgcn_rsqf(r2);
                const float r = r2 * ir;
                const float w = 1.f - r * __builtin_amdgcn_rcpf(a.dy.dpd_rc);
                const float ex = -dx * ir, ey = -dy * ir, ez = -dz * ir;
                // v_i - (v_j - s shear_rate Ly e_x)
                const float vx = vi.x - vj.x + (float)(s * g.le_rate_Ly);
                const float vy = vi.y - vj.y;
                const float vz = vi.z - vj.z;
                const float ev = ex * vx + ey * vy + ez * vz;
                const float th = dpd_theta(a.dy.seed, (uint64_t)step, __float_as_uint(vi.w), __float_as_uint(vj.w));
                const float A = -a.dy.dpd_gamma * w * w * ev + a.dy.dpd_sigma_isdt * w * th;
                fx += A * ex;
                fy += A * ey;
                fz += A * ez;
            }
        }
        acc[A_EPAIR] += 0.5 * (double)ue;
        acc[A_VIR] += 0.5 * (double)we;
        if (tensor) {
            acc[A_TXX] += 0.5 * (double)txx; acc[A_TYY] += 0.5 * (double)tyy; acc[A_TZZ] += 0.5 * (double)tzz;
            acc[A_TXY] += 0.5 * (double)txy; acc[A_TXZ] += 0.5 * (double)txz; acc[A_TYZ] += 0.5 * (double)tyz;
        }
        if (BONDED) {
            const auto dfb = [&df](const int4& p, const int4& q, float& ddx, float& ddy, float& ddz) {
                (void)df(p, q, ddx, ddy, ddz);
            };
            bonded_forces<float, int4, decltype(dfb), true>(b, a.dy, n, i, xq, qi, dfb, fx, fy, fz, acc, tensor,
                                                            flag_bond);
        }
        const double F[3] = {(double)fx, (double)fy, (double)fz};
        finish_particle(a, i, xi, ti, F, acc, flag_reb, flag_nf, g.le ? &les : nullptr);
    }
    block_epilogue<BS>(a, acc, flag_reb, flag_bond, flag_nf, tensor ? kNacc : kNaccStep, blk, grid);
}

// The DPD step of one particle type (k_step_gen's terms in its order, some
// contracted otherwise; MODE_STEP, without AdResS), sheared (LE) or not.  Drawing theta_ij costs ten rounds of quarter-
// rate multiplies, and the lanes of a wavefront draw together: walking the list
// with the draw inside spends it on nearly every slot, though less than half
// of a lane's slots are within the cutoffs ((1 / 1.3)^3 at skin 0.3).  So each
// lane first collects the neighbours within the larger cutoff in LDS (kDpdQueue
// of them at a time) and the forces walk what it collected, in list order.
// Bound by VALU issue: 1,048,576 particles at density 3 under shear, step kernel
// 245 -> 190 us.
constexpr int kDpdQueue = 32;
template <bool BONDED, bool LE, int BS>
__global__ void __launch_bounds__(BS) k_step_dpd(const StepArgs a) {
    extern __shared__ float2 stab[];
    __shared__ int32_t queue[BS / 64][kDpdQueue][64];
    int blk, grid;
    if (finalize_block<BS>(a, blk, grid)) return;
    const Geom& g = a.g;
    const Bufs& b = a.b;
    const int64_t n = g.n;
    const int4* __restrict__ xq = b.xq[a.parity];
    const double4* __restrict__ x64 = b.x[a.parity];
    const float4* __restrict__ vs = reinterpret_cast<const float4*>(b.vt);
    const int ntab = a.pt.tabn[0];
    if (ntab > 1) {
        for (int k = threadIdx.x; k < ntab; k += BS) stab[k] = b.tab[k];
        __syncthreads();
    }
    double acc[kNacc];
#pragma unroll
    for (int k = 0; k < kNacc; ++k) acc[k] = 0.0;
    bool flag_reb = false, flag_bond = false, flag_nf = false;
    const bool tensor = a.tensor != 0;
    const int64_t step = b.ctl->step;
    double dw = 0.0;
    uint32_t qd = 0;
    LeStep les{0.0, 0.0};
    if (LE) {
        const double delta = le_delta(g, step);
        dw = le_fold(g, delta);
        qd = quantize(delta, g.qs[0]);
        les.delta_next = le_delta(g, step + 1);
        les.drift = fabs(g.le_rate_Ly * ((double)(step + 1 - b.ctl->build_step) * g.le_dt));
    }
    const int64_t i = (int64_t)xcd_block(blk, grid) * BS + threadIdx.x;
    if (i < n) {
        const int lane = threadIdx.x & 63;
        int32_t(*const qu)[64] = queue[threadIdx.x >> 6];
        const double4 xi = x64[i];
        const int4 qi = quantize4(g, xi.x, xi.y, xi.z, xi.w);
        const float4 vi = vs[i];
        const DiffLEQ df{g.ql[0], g.ql[1], g.ql[2], qd};
        // a wavefront with no particle within the list radius of the sheared
        // boundary meets no displaced image
        // (a thousandth more than that, for the coordinates' rounding)
        const double rv = 1.001 * sqrt(g.rv2);
        const bool edge = LE && __any(xi.y < rv || xi.y > g.L[1] - rv);
        auto diff = [&](const int4& qj, float& dx, float& dy, float& dz) __attribute__((always_inline)) {
            if (edge) return df(qi, qj, dx, dy, dz);
            dx = qdiff(qj.x, qi.x, g.ql[0]);
            dy = qdiff(qj.y, qi.y, g.ql[1]);
            dz = qdiff(qj.z, qi.z, g.ql[2]);
            return 0;
        };
        const float rc2lo = a.pt.rc2lo[0], rc2hi = a.pt.rc2hi[0], dpd_rc2 = a.dy.dpd_rc2;
        const float reach2 = fmaxf(rc2hi, dpd_rc2);
        const float irc = __builtin_amdgcn_rcpf(a.dy.dpd_rc);
        float fx = 0.f, fy = 0.f, fz = 0.f, ue = 0.f, we = 0.f;
        float txx = 0.f, tyy = 0.f, tzz = 0.f, txy = 0.f, txz = 0.f, tyz = 0.f;
        int qn = 0;
        // the collected neighbours, the next one's record and velocity ahead
        auto forces = [&]() __attribute__((always_inline)) {
            __builtin_amdgcn_wave_barrier();
            int jn = qn > 0 ? qu[0][lane] : (int)i;
            int4 qnx = xq[jn];
            float4 vn = vs[jn];
            for (int t = 0; t < qn; ++t) {
                const int j = jn;
                const int4 qj = qnx;
                const float4 vj = vn;
                jn = qu[min(t + 1, qn - 1)][lane];
                qnx = xq[jn];
                vn = vs[jn];
                float dx, dy, dz;
                const int s = diff(qj, dx, dy, dz);
                const float r2 = dx * dx + dy * dy + dz * dz;
                bool in = r2 < rc2lo;
                if (!in && r2 < rc2hi) in = exact_r2_le(g, xi, x64[j], dw) < a.pt.rc2d[0];
                if (in) {
                    const PairCoef<float>& c = a.pt.f[0];
                    float fr, u;
                    if (ntab > 1) {
                        const float r = sqrtf(r2);
                        float q = (r - a.pt.tab_rmin[0]) * a.pt.tab_idr[0];
                        q = q > 0.f ? q : 0.f;
                        int kq = (int)q;
                        kq = kq > ntab - 2 ? ntab - 2 : kq;
                        const float al = q - (float)kq;
                        const float2 t0 = stab[kq], t1 = stab[kq + 1];
                        u = (1.f - al) * t0.x + al * t1.x;
                        fr = ((1.f - al) * t0.y + al * t1.y) * __builtin_amdgcn_rcpf(r);
                    } else if (c.cap2 > 0.f && r2 < c.cap2) {
                        fr = c.fcap * __builtin_amdgcn_rsqf(r2);
                        u = c.ucap;
                    } else {
                        const float inv = __builtin_amdgcn_rcpf(r2);
                        const float s2 = c.sig2 * inv;
                        const float s6 = s2 * s2 * s2;
                        fr = c.eps24 * s6 * (2.f * s6 - 1.f) * inv;
                        u = c.eps4 * s6 * (s6 - 1.f) - c.shift;
                    }
                    fx -= fr * dx;
                    fy -= fr * dy;
                    fz -= fr * dz;
                    ue += u;
                    we += fr * r2;
                    if (tensor) {
                        txx += fr * dx * dx; tyy += fr * dy * dy; tzz += fr * dz * dz;
                        txy += fr * dx * dy; txz += fr * dx * dz; tyz += fr * dy * dz;
                    }
                }
                if (r2 < dpd_rc2 && r2 > 0.f) {
                    const float ir = __builtin_amdgcn_rsqf(r2);
                    const float r = r2 * ir;
                    const float w = 1.f - r * irc;
                    const float ex = -dx * ir, ey = -dy * ir, ez = -dz * ir;
                    // v_i - (v_j - s shear_rate Ly e_x)
                    const float vx = vi.x - vj.x + (float)(s * g.le_rate_Ly);
                    const float vy = vi.y - vj.y;
                    const float vz = vi.z - vj.z;
                    const float ev = ex * vx + ey * vy + ez * vz;
                    const float th = dpd_theta(a.dy.seed, (uint64_t)step, __float_as_uint(vi.w), __float_as_uint(vj.w));
                    const float A = -a.dy.dpd_gamma * w * w * ev + a.dy.dpd_sigma_isdt * w * th;
                    fx += A * ex;
                    fy += A * ey;
                    fz += A * ez;
                }
            }
            __builtin_amdgcn_wave_barrier();
            qn = 0;
        };
        int cnt = b.ncount[i];
        cnt = cnt < g.cap ? cnt : g.cap;
        const int nslots = min((cnt + 7) & ~7, g.cap);   // padded with the particle itself
        const int32_t* __restrict__ row = b.nl + nl_base(i, g.cap);
        constexpr int B = 8;
        const int last = nslots > 0 ? nslots - 1 : 0;
        int jn[B];
#pragma unroll
        for (int u = 0; u < B; ++u) jn[u] = nslots > 0 ? row[nl_off(u)] : (int)i;
        for (int k0 = 0; k0 < nslots; k0 += B) {
            int jc[B];
            int4 q[B];
#pragma unroll
            for (int u = 0; u < B; ++u) {
                jc[u] = jn[u];
                q[u] = xq[jc[u]];
            }
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const int kk = k0 + B + u;
                jn[u] = row[nl_off(kk < last ? kk : last)];
            }
            if (__any(qn > kDpdQueue - B)) forces();
#pragma unroll
            for (int u = 0; u < B; ++u) {
                float dx, dy, dz;
                (void)diff(q[u], dx, dy, dz);
                const float r2 = dx * dx + dy * dy + dz * dz;
                qu[qn][lane] = jc[u];
                qn += (k0 + u < cnt && r2 < reach2) ? 1 : 0;
            }
        }
        forces();
        acc[A_EPAIR] += 0.5 * (double)ue;
        acc[A_VIR] += 0.5 * (double)we;
        if (tensor) {
            acc[A_TXX] += 0.5 * (double)txx; acc[A_TYY] += 0.5 * (double)tyy; acc[A_TZZ] += 0.5 * (double)tzz;
            acc[A_TXY] += 0.5 * (double)txy; acc[A_TXZ] += 0.5 * (double)txz; acc[A_TYZ] += 0.5 * (double)tyz;
        }
        if (BONDED) {
            const auto dfb = [&df](const int4& p, const int4& q, float& ddx, float& ddy, float& ddz) {
                (void)df(p, q, ddx, ddy, ddz);
            };
            bonded_forces<float, int4, decltype(dfb), true>(b, a.dy, n, i, xq, qi, dfb, fx, fy, fz, acc, tensor,
                                                            flag_bond);
        }
        const double F[3] = {(double)fx, (double)fy, (double)fz};
        finish_particle(a, i, xi, 0, F, acc, flag_reb, flag_nf, LE ? &les : nullptr);
    }
    block_epilogue<BS>(a, acc, flag_reb, flag_bond, flag_nf, tensor ? kNacc : kNaccStep, blk, grid);
}

// The AdResS step of one particle type without shear or DPD (k_step_gen's
// terms in its order; the mix is contracted otherwise, so forces differ in
// rounding, about 1e-6 of the largest), the pair and coarse-grained tables in
// LDS.  Bound by VALU issue
// and the texture-data path together.  Records are gathered four at a time and
// the registers held to five wavefronts per SIMD: 299,997 particles are 4,688
// wavefronts, which four per SIMD (4,096 on the card) run in two rounds.  Step
// kernel at that size, density 0.8442: k_step_gen 125 us; here 104 us with four
// per SIMD and eight records, 101 with five and eight, 89-92 with five and
// four.  20 steps with their list builds, this tree against the generic kernel
// and the builds before it: 1.74x at 4,000 particles, 1.40x at 60,000, 1.31x at
// 150,000, 1.28x at 500,000, 1.38x at 1,000,000.  Leaving out the force of weight 0 in wavefronts that need one force
// only gained 2 us and was not worth three copies of the loop.
template <bool BONDED, int BS>
__global__ void __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(5))) k_step_adress(const StepArgs a) {
    extern __shared__ float2 stab[];
    int blk, grid;
    if (finalize_block<BS>(a, blk, grid)) return;
    const Geom& g = a.g;
    const Bufs& b = a.b;
    const int64_t n = g.n;
    const int4* __restrict__ xq = b.xq[a.parity];
    const double4* __restrict__ x64 = b.x[a.parity];
    const int np = g.table_points;
    {
        const float2* __restrict__ src0 = b.tab;
        const float2* __restrict__ src1 = b.tab + (int64_t)kCgTableRow * np;
        for (int k = threadIdx.x; k < np; k += BS) {
            stab[k] = src0[k];
            stab[np + k] = src1[k];
        }
        __syncthreads();
    }
    double acc[kNacc];
#pragma unroll
    for (int k = 0; k < kNacc; ++k) acc[k] = 0.0;
    bool flag_reb = false, flag_bond = false, flag_nf = false;
    const bool tensor = a.tensor != 0;
    const int64_t i = (int64_t)xcd_block(blk, grid) * BS + threadIdx.x;
    if (i < n) {
        const double4 xi = x64[i];
        const int4 qi = quantize4(g, xi.x, xi.y, xi.z, xi.w);
        const float Lx = (float)g.L[0];
        const float rc2lo = a.pt.rc2lo[0], rc2hi = a.pt.rc2hi[0];
        const int cgn = a.pt.cgn[0], ntab = a.pt.tabn[0];
        const float cg_rc2lo = cgn > 1 ? a.pt.cg_rc2lo[0] : 0.f, cg_rc2hi = cgn > 1 ? a.pt.cg_rc2hi[0] : 0.f;
        const PairCoef<float>& c = a.pt.f[0];
        const float wi = adress_weight(a.dy, (float)xi.x, Lx);
        float fx = 0.f, fy = 0.f, fz = 0.f, ue = 0.f, we = 0.f;
        float txx = 0.f, tyy = 0.f, tzz = 0.f, txy = 0.f, txz = 0.f, tyz = 0.f;
        int cnt = b.ncount[i];
        cnt = cnt < g.cap ? cnt : g.cap;
        const int nslots = min((cnt + 7) & ~7, g.cap);   // padded with the particle itself
        const int32_t* __restrict__ row = b.nl + nl_base(i, g.cap);
        // u and f = -du/dr of a row of np points, linear in r
        auto lookup = [&](const float2* t, int nt, float rmin, float idr, float r, float& u,
                          float& fr) __attribute__((always_inline)) {
            float q = (r - rmin) * idr;
            q = q > 0.f ? q : 0.f;
            int kq = (int)q;
            kq = kq > nt - 2 ? nt - 2 : kq;
            const float al = q - (float)kq;
            const float2 t0 = t[kq], t1 = t[kq + 1];
            u = (1.f - al) * t0.x + al * t1.x;
            fr = ((1.f - al) * t0.y + al * t1.y) * __builtin_amdgcn_rcpf(r);
        };
        constexpr int B = 4;
        const int last = nslots > 0 ? nslots - 1 : 0;
        int jn[B];
#pragma unroll
        for (int u = 0; u < B; ++u) jn[u] = nslots > 0 ? row[nl_off(u)] : (int)i;
        for (int k0 = 0; k0 < nslots; k0 += B) {
            int jc[B];
            int4 q[B];
#pragma unroll
            for (int u = 0; u < B; ++u) {
                jc[u] = jn[u];
                q[u] = xq[jc[u]];
            }
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const int kk = k0 + B + u;
                jn[u] = row[nl_off(kk < last ? kk : last)];
            }
#pragma unroll
            for (int v = 0; v < B; ++v) {
                const float dx = qdiff(q[v].x, qi.x, g.ql[0]);
                const float dy = qdiff(q[v].y, qi.y, g.ql[1]);
                const float dz = qdiff(q[v].z, qi.z, g.ql[2]);
                const float r2 = dx * dx + dy * dy + dz * dz;
                const bool ok = k0 + v < cnt;
                bool in = ok && r2 < rc2lo;
                bool cg = ok && r2 < cg_rc2lo;
                if (ok && !in && r2 < rc2hi) in = exact_r2_le(g, xi, x64[jc[v]], 0.0) < a.pt.rc2d[0];
                if (ok && !cg && r2 < cg_rc2hi) cg = exact_r2_le(g, xi, x64[jc[v]], 0.0) < a.pt.cg_rc2d[0];
                if (!in && !cg) continue;
                float ucg = 0.f, frcg = 0.f, fr = 0.f, u = 0.f;
                if (cg) lookup(stab + np, cgn, a.pt.cg_rmin[0], a.pt.cg_idr[0], sqrtf(r2), ucg, frcg);
                if (!in) {
                } else if (ntab > 1) {
                    lookup(stab, ntab, a.pt.tab_rmin[0], a.pt.tab_idr[0], sqrtf(r2), u, fr);
                } else if (c.cap2 > 0.f && r2 < c.cap2) {
                    fr = c.fcap * __builtin_amdgcn_rsqf(r2);
                    u = c.ucap;
                } else {
                    const float inv = __builtin_amdgcn_rcpf(r2);
                    const float s2 = c.sig2 * inv;
                    const float s6 = s2 * s2 * s2;
                    fr = c.eps24 * s6 * (2.f * s6 - 1.f) * inv;
                    u = c.eps4 * s6 * (s6 - 1.f) - c.shift;
                }
                // x_j from its fixed-point coordinate (positions lie in [0, L))
                const float lam = wi * adress_weight(a.dy, (float)(uint32_t)q[v].x * g.ql[0], Lx);
                u = lam * u + (1.f - lam) * ucg;
                fr = lam * fr + (1.f - lam) * frcg;
                fx -= fr * dx;
                fy -= fr * dy;
                fz -= fr * dz;
                ue += u;
                we += fr * r2;
                if (tensor) {
                    txx += fr * dx * dx; tyy += fr * dy * dy; tzz += fr * dz * dz;
                    txy += fr * dx * dy; txz += fr * dx * dz; tyz += fr * dy * dz;
                }
            }
        }
        acc[A_EPAIR] += 0.5 * (double)ue;
        acc[A_VIR] += 0.5 * (double)we;
        if (tensor) {
            acc[A_TXX] += 0.5 * (double)txx; acc[A_TYY] += 0.5 * (double)tyy; acc[A_TZZ] += 0.5 * (double)tzz;
            acc[A_TXY] += 0.5 * (double)txy; acc[A_TXZ] += 0.5 * (double)txz; acc[A_TYZ] += 0.5 * (double)tyz;
        }
        if (BONDED) {
            const DiffLEQ df{g.ql[0], g.ql[1], g.ql[2], 0u};
            const auto dfb = [&df](const int4& p, const int4& q, float& ddx, float& ddy, float& ddz) {
                (void)df(p, q, ddx, ddy, ddz);
            };
            bonded_forces<float, int4, decltype(dfb), true>(b, a.dy, n, i, xq, qi, dfb, fx, fy, fz, acc, tensor,
                                                            flag_bond);
        }
        const double F[3] = {(double)fx, (double)fy, (double)fz};
        finish_particle(a, i, xi, 0, F, acc, flag_reb, flag_nf, nullptr);
    }
    block_epilogue<BS>(a, acc, flag_reb, flag_bond, flag_nf, tensor ? kNacc : kNaccStep, blk, grid);
}

// Step of the surrogate mode, one 256-particle tile per block: the
// network's pair force from the per-particle input gradients a_i = dE_i/dG(i),
//   F_i = sum_j ((a_i + a_j) . g'(r_ij)) (x_j - x_i) / r_ij  over r_ij < r_d,
//   g'_k(r) = phi_k(r) (f_c'(r) - (r - mu_k) f_c(r) / w^2),
// then the bonded forces, the integration and the reductions of the plain
// step kernels.  The list row is pipelined: positions are gathered two slots
// ahead and the a_j rows of in-range neighbours one slot ahead of the pair
// arithmetic that uses them.  BF16 form (A16): a rows are
// BF16; g' is rounded to BF16 pairs and dotted with a_i and a_j by
// v_dot2_f32_bf16 with FP32 accumulation.  FP32 form: the pair force, its
// virial and tensor come from the pass before (s.f, s.u).  The pair virial goes
// to the step's reductions; the network energy comes from the network
// kernel's partials.
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));

template <bool BONDED, bool TENSOR, bool A16>
__global__ void __launch_bounds__(kBlock) k_sur_step(const StepArgs a, const SurBufs s, const SurConst c) {
    int blk, grid;
    if (finalize_block(a, blk, grid)) return;
    constexpr int AW = 16;                  // 32-bit words per a row
    const Geom& g = a.g;
    const Bufs& b = a.b;
    const int64_t n = g.n;
    double acc[kNacc];
#pragma unroll
    for (int k = 0; k < kNacc; ++k) acc[k] = 0.0;
    bool flag_reb = false, flag_bond = false, flag_nf = false;
    const int64_t i = (int64_t)xcd_block(blk, grid) * kBlock + threadIdx.x;
    if (i < n) {
        const int4* __restrict__ xq = b.xq[a.parity];
        const double4 xi = b.x[a.parity][i];
        const int4 qi = quantize4(g, xi.x, xi.y, xi.z, xi.w);
        float fx = 0.f, fy = 0.f, fz = 0.f, wv = 0.f;
        float txx = 0.f, tyy = 0.f, tzz = 0.f, txy = 0.f, txz = 0.f, tyz = 0.f;
        if (!A16) {
            const float4 f = s.f[i];
            fx = f.x; fy = f.y; fz = f.z; wv = f.w;
            if (TENSOR) {
                const float* t = s.u + i * kSurNB;
                txx = t[0]; tyy = t[1]; tzz = t[2]; txy = t[3]; txz = t[4]; tyz = t[5];
            }
        } else {
        const uint32_t* __restrict__ arow = reinterpret_cast<const uint32_t*>(s.ab);
        uint32_t ai[AW];
#pragma unroll
        for (int q = 0; q < AW / 4; ++q) {
            const uint4 v = reinterpret_cast<const uint4*>(arow + i * AW)[q];
            ai[4 * q] = v.x; ai[4 * q + 1] = v.y; ai[4 * q + 2] = v.z; ai[4 * q + 3] = v.w;
        }
        int cnt = b.ncount[i];
        cnt = cnt < g.cap ? cnt : g.cap;
        const int nslots = min((cnt + 7) & ~7, g.cap);
        const int32_t* __restrict__ row = b.nl + nl_base(i, g.cap);
        const int last = nslots > 0 ? nslots - 1 : 0;
        auto idx = [&](int slot) { return row[nl_off(slot < last ? slot : last)]; };
        auto geom = [&](const int4& qj, float& dx, float& dy, float& dz) {
            dx = qdiff(qj.x, qi.x, g.ql[0]);
            dy = qdiff(qj.y, qi.y, g.ql[1]);
            dz = qdiff(qj.z, qi.z, g.ql[2]);
            return dx * dx + dy * dy + dz * dz;
        };
        auto load_row = [&](int j, uint32_t* out) {
#pragma unroll
            for (int q = 0; q < AW / 4; ++q) {
                const uint4 v = reinterpret_cast<const uint4*>(arow + (int64_t)j * AW)[q];
                out[4 * q] = v.x; out[4 * q + 1] = v.y; out[4 * q + 2] = v.z; out[4 * q + 3] = v.w;
            }
        };
        auto pair = [&](const int4& qj, const uint32_t* aj) {
            float dx, dy, dz;
            const float r2 = geom(qj, dx, dy, dz);
            const float r = sqrtf(r2);
            float dfc;
            const float fc = sur_cutoff(c, r, dfc);
            float ph[kSurNB];
            sur_basis(c, r, ph);
            const float Bc = c.inv_w2 * fc;
            float cij = 0.f;
            {
                // g'_k = phi_k (dfc - (r - mu_k) Bc) = phi_k (mu_k Bc + al): one
                // FMA and one product per term (the FP32 cancellation of
                // mu_k Bc against al is far below the BF16 rounding that follows)
                const float al = fmaf(-r, Bc, dfc);
#pragma unroll
                for (int k2 = 0; k2 < kSurNB / 2; ++k2) {
                    const float g0 = ph[2 * k2] * fmaf(c.mu[2 * k2], Bc, al);
                    const float g1 = ph[2 * k2 + 1] * fmaf(c.mu[2 * k2 + 1], Bc, al);
                    const bf16x2v gp = {(__bf16)g0, (__bf16)g1};
                    cij = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2v, ai[k2]), gp, cij, false);
                    cij = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2v, aj[k2]), gp, cij, false);
                }
            }
            const float sc = cij * __builtin_amdgcn_rcpf(r);
            fx += sc * dx;
            fy += sc * dy;
            fz += sc * dz;
            wv -= cij * r;
            if (TENSOR) {
                // r_ij f_ij with r_ij = -(dx, dy, dz), f_ij = sc (dx, dy, dz)
                txx -= sc * dx * dx; tyy -= sc * dy * dy; tzz -= sc * dz * dz;
                txy -= sc * dx * dy; txz -= sc * dx * dz; tyz -= sc * dy * dz;
            }
        };
        auto in_range = [&](const int4& qj) {
            float dx, dy, dz;
            const float r2 = geom(qj, dx, dy, dz);
            return r2 < c.rd2 && r2 > 0.f;   // r2 = 0: the row's padding (the particle itself)
        };
        if (nslots > 0) {
            // slot k: index jA, position qA, a row aX (in range: inX); slot k+1:
            // index jB, position qB (in flight); slot k+2: index jC.  Rows hold
            // a multiple of 8 slots, so slots come in pairs and the a rows
            // alternate between aX and aY without copies.
            int jA = idx(0), jB = idx(1), jC = idx(2);
            int4 qA = xq[jA], qB = xq[jB];
            uint32_t aX[AW], aY[AW];
            bool inX = in_range(qA), inY = false;
            if (inX) load_row(jA, aX);
            for (int k0 = 0; k0 < nslots; k0 += 2) {
                // slot k0 (row aX); prefetch: a row of k0 + 1, position of k0 + 2
                inY = in_range(qB);
                if (inY) load_row(jB, aY);
                int4 qC = xq[jC];
                int jD = idx(k0 + 3);
                if (inX) pair(qA, aX);
                qA = qB; qB = qC; jA = jB; jB = jC; jC = jD;
                // slot k0 + 1 (row aY); prefetch: a row of k0 + 2, position of k0 + 3
                inX = k0 + 2 < nslots && in_range(qB);
                if (inX) load_row(jB, aX);
                qC = xq[jC];
                jD = idx(k0 + 4);
                if (inY) pair(qA, aY);
                qA = qB; qB = qC; jA = jB; jB = jC; jC = jD;
            }
        }
        }
        acc[A_VIR] += 0.5 * (double)wv;
        if (TENSOR) {
            acc[A_TXX] += 0.5 * (double)txx; acc[A_TYY] += 0.5 * (double)tyy; acc[A_TZZ] += 0.5 * (double)tzz;
            acc[A_TXY] += 0.5 * (double)txy; acc[A_TXZ] += 0.5 * (double)txz; acc[A_TYZ] += 0.5 * (double)tyz;
        }
        if (BONDED) {
            const DiffQ df{g.ql[0], g.ql[1], g.ql[2]};
            bonded_forces<float, int4, DiffQ>(b, a.dy, n, i, xq, qi, df, fx, fy, fz, acc, TENSOR, flag_bond);
        }
        const double F[3] = {(double)fx, (double)fy, (double)fz};
        finish_particle(a, i, xi, (int)xi.w, F, acc, flag_reb, flag_nf);
    }
    block_epilogue(a, acc, flag_reb, flag_bond, flag_nf, TENSOR ? kNacc : kNaccStep, blk, grid);
}

// ------------------------------------------------------------------ batches
//
// Per-tile kernels of a batch: block -> global tile (XCD-aware order) ->
// system -> the single-system body on that system's arrays.  The rebuild
// kernels return at once for systems whose own rebuild flag is clear.

struct TileRef {
    const SysEntry* e;
    int64_t lt;     // tile inside the system
    int64_t i;      // particle inside the system
};

__device__ __forceinline__ TileRef tile_ref(const SysEntry* __restrict__ tab, const int32_t* __restrict__ tile_sys) {
    const int64_t t = xcd_block(blockIdx.x, gridDim.x);
    const SysEntry* e = tab + tile_sys[t];
    const int64_t lt = t - e->tile0;
    return TileRef{e, lt, lt * kBlock + threadIdx.x};
}

// Rebuild kernels of a batch take the plain block order instead: only the
// members whose own trigger fired have work, and the XCD-contiguous order
// would put all of a rebuilding member's tiles on one XCD while the others
// idle.  Spread round-robin, every member's tiles use all XCDs (measured: the
// 256-replica batch 3.62e9 -> 4.15e9 atom-steps/s).
__device__ __forceinline__ TileRef tile_ref_spread(const SysEntry* __restrict__ tab,
                                                   const int32_t* __restrict__ tile_sys) {
    const int64_t t = blockIdx.x;
    const SysEntry* e = tab + tile_sys[t];
    const int64_t lt = t - e->tile0;
    return TileRef{e, lt, lt * kBlock + threadIdx.x};
}

// Starts every member's step (advance) and asks whether any rebuilds.
__global__ void k_batch_any(BatchCells bc, int parity, int advance) {
    __shared__ int any;
    if (threadIdx.x == 0) any = 0;
    __syncthreads();
    for (int s = threadIdx.x; s < bc.nsys; s += blockDim.x) {
        const Bufs& b = bc.tab[s].a.b;
        if (advance) advance_step(b, parity);
        if (rebuild_requested(b, parity)) any = 1;
    }
    __syncthreads();
    if (threadIdx.x == 0) bc.gb.ctl->rebuild[0] = (uint32_t)any;
}

__global__ void __launch_bounds__(kBlock) k_batch_bin(const SysEntry* __restrict__ tab,
                                                      const int32_t* __restrict__ tile_sys, int parity) {
    const TileRef r = tile_ref_spread(tab, tile_sys);
    const Bufs& b = r.e->a.b;
    if (!rebuild_requested(b, parity)) return;
    const Geom& g = r.e->a.g;
    bin_one(g, b, r.i, r.i < g.n, parity);
}

// prefix of the concatenated counts at each system's first cell
__global__ void k_batch_bases(BatchCells bc) {
    if (!rebuild_requested(bc.gb, 0)) return;
    for (int s = threadIdx.x; s < bc.nsys; s += blockDim.x) bc.base[s] = bc.gb.cstart[bc.c_off[s]];
}

// cell starts of rebuilding systems become offsets inside the system
__global__ void __launch_bounds__(kBlock) k_batch_localize(BatchCells bc, int parity) {
    if (!rebuild_requested(bc.gb, 0)) return;
    for (int64_t c = gtid(); c < bc.gg.ncell; c += gstride()) {
        int lo = 0, hi = bc.nsys;   // system with c_off[s] <= c < c_off[s + 1]
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (bc.c_off[mid] <= c) lo = mid; else hi = mid;
        }
        if (rebuild_requested(bc.tab[lo].a.b, parity)) bc.gb.cstart[c] -= bc.base[lo];
    }
}

__global__ void __launch_bounds__(kBlock) k_batch_scatter(const SysEntry* __restrict__ tab,
                                                          const int32_t* __restrict__ tile_sys, int parity) {
    const TileRef r = tile_ref_spread(tab, tile_sys);
    const Bufs& b = r.e->a.b;
    if (!rebuild_requested(b, parity)) return;
    scatter_one(r.e->a.g, b, r.i, r.i < r.e->a.g.n, parity);
}

__global__ void __launch_bounds__(kBlock) k_batch_rank(const SysEntry* __restrict__ tab,
                                                       const int32_t* __restrict__ tile_sys, int parity) {
    const TileRef r = tile_ref_spread(tab, tile_sys);
    const Bufs& b = r.e->a.b;
    if (!rebuild_requested(b, parity)) return;
    if (r.i < r.e->a.g.n) rank_one(r.e->a.g, b, r.i, parity, r.e->bonded);
}

// The members' lists, one wavefront per 64 particles (four to a tile of the
// batch): on the matrix cores or one particle per lane, by member.  Both in
// one launch: a batch's build lasts as long as its slowest wavefront, in two
// launches as long as the sum of theirs (48 LJ members of 600 to 1,540
// particles, some too small for the matrix cores, 40 steps: 15.5 ms in two
// launches, 12.0 in one).
union NlBatch {
    NlWave mat;
    int32_t rows[kNlLds + 1][64];
};
__global__ void __launch_bounds__(kTile) k_batch_nl(const SysEntry* __restrict__ tab,
                                                    const int32_t* __restrict__ tile_sys, int parity) {
    __shared__ NlBatch sh;
    const SysEntry* e = tab + tile_sys[blockIdx.x / (kBlock / kTile)];
    const Bufs& b = e->a.b;
    const Geom& g = e->a.g;
    if (!rebuild_requested(b, parity)) return;
    const int64_t t = (int64_t)blockIdx.x - e->tile0 * (kBlock / kTile);
    if (t * kTile >= g.n) return;
    int local_max = 0;
    bool overflow = false;
    if (g.nl_mat) {
        nl_mtile<false>(g, b, t, parity, e->bonded, sh.mat, LeNl{0.0, 0.0, 0u}, local_max, overflow);
    } else {
        const int64_t i = t * kTile + threadIdx.x;
        if (i < g.n) nl_one(g, b, i, parity, e->bonded, sh.rows, local_max, overflow);
    }
    nl_epilogue(b, local_max, overflow);
}

// Fused force + integrate for one tile of one system (FP32 fast path: one
// particle type, cubic box, no capping radius), partials at the tile's slot.
// The table holds each system's arguments for one (mode, parity); they are
// read in place, never copied.
// Capped at 128 VGPRs like the bonded single-system kernel (the batch holds
// melts): 637 -> 615 us per step for the 256-replica batch.
template <bool TENSOR>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4)))
k_batch_step(const SysEntry* __restrict__ tab, const int32_t* __restrict__ tile_sys) {
    const TileRef r = tile_ref(tab, tile_sys);
    const StepArgs& a = r.e->a;
    double acc[kNacc];
#pragma unroll
    for (int k = 0; k < kNacc; ++k) acc[k] = 0.0;
    bool flag_reb = false, flag_bond = false, flag_nf = false;
    if (r.i < a.g.n) {
        if (r.e->bonded) fast_particle<true, TENSOR>(a, r.i, acc, flag_reb, flag_bond, flag_nf);
        else fast_particle<false, TENSOR>(a, r.i, acc, flag_reb, flag_bond, flag_nf);
    }
    block_epilogue(a, acc, flag_reb, flag_bond, flag_nf, TENSOR ? kNacc : kNaccStep, r.lt, r.e->ntiles);
}

__global__ void __launch_bounds__(kFinal) k_batch_observe(const SysEntry* __restrict__ tab) {
    const SysEntry& e = tab[blockIdx.x];
    finalize_body<kFinal, kNacc>(e.a.b, e.a.parity, e.ntiles, MODE_OBSERVE, nullptr);
}

// The end of a call's last step.  Members keep no per-step records (a batch has
// no history call), so only the counters move.
__global__ void k_batch_end(BatchCells bc) {
    for (int s = threadIdx.x; s < bc.nsys; s += blockDim.x) {
        DevCtl* c = bc.tab[s].a.b.ctl;
        c->step += 1;
        c->vel_half = 1;
        c->ran = 0;
    }
}

__global__ void k_batch_gather_obs(const SysEntry* __restrict__ tab, int nsys, double* out) {
    for (int k = threadIdx.x; k < nsys * kHistRec; k += blockDim.x) out[k] = tab[k / kHistRec].a.b.cur[k % kHistRec];
}

// ------------------------------------------------------------------ launchers

static inline int grid_for(int64_t n, int cap_blocks = 4096) {
    int64_t g = (n + kBlock - 1) / kBlock;
    if (g < 1) g = 1;
    if (g > cap_blocks) g = cap_blocks;
    return (int)g;
}

// One 256-particle tile per block: with about three resident blocks per CU a
// capped grid of multi-tile blocks leaves a partial second wave; single-tile
// blocks let the dispatcher balance the tail (measured: 8 % faster for the
// LJ fluid, 19 % for the melt than 1,024 blocks of 4 tiles).
int step_grid(int64_t n) {
    const int64_t t = (n + kBlock - 1) / kBlock;
    return (int)(t < 1 ? 1 : t);
}

hipError_t launch_init_load(const Geom& g, const Bufs& b, int parity, const double* pos,
                            const double* vel, const int32_t* type, const int32_t* image,
                            hipStream_t s) {
    hipLaunchKernelGGL(k_init_load, dim3(grid_for(g.n)), dim3(kBlock), 0, s, g, b, parity, pos, vel, type,
                       image);
    return hipGetLastError();
}

hipError_t launch_overwrite_state(const Geom& g, const Bufs& b, int parity, const double* pos,
                                  const double* vel, const int32_t* image, hipStream_t s) {
    hipLaunchKernelGGL(k_overwrite_state, dim3(grid_for(g.n)), dim3(kBlock), 0, s, g, b, parity, pos, vel,
                       image);
    return hipGetLastError();
}

hipError_t launch_get_state(const Geom& g, const Bufs& b, int parity, double* pos, double* vel,
                            int32_t* image, double* pos_build, hipStream_t s) {
    hipLaunchKernelGGL(k_get_state, dim3(grid_for(g.n)), dim3(kBlock), 0, s, g, b, parity, pos, vel, image,
                       pos_build);
    return hipGetLastError();
}

hipError_t launch_get_neighbors(const Geom& g, const Bufs& b, int32_t* count, int32_t* idx, int32_t cap,
                                hipStream_t s) {
    hipLaunchKernelGGL(k_get_neighbors, dim3(grid_for(g.n)), dim3(kBlock), 0, s, g, b, count, idx, cap);
    return hipGetLastError();
}

hipError_t launch_set_ctl(const Bufs& b, int64_t step, int vel_half, int rebuild, int clear_status,
                          hipStream_t s) {
    hipLaunchKernelGGL(k_set_ctl, dim3(1), dim3(64), 0, s, b, step, vel_half, rebuild, clear_status);
    return hipGetLastError();
}

hipError_t launch_zero_i32(int32_t* p, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_zero_i32, dim3(grid_for(n)), dim3(kBlock), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_copy_i32(int32_t* dst, const int32_t* src, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_copy_i32, dim3(grid_for(n)), dim3(kBlock), 0, s, dst, src, n);
    return hipGetLastError();
}

hipError_t launch_clear_rebuild(const Bufs& b, hipStream_t s) {
    hipLaunchKernelGGL(k_clear_rebuild, dim3(1), dim3(64), 0, s, b);
    return hipGetLastError();
}

hipError_t launch_rebuild(const Geom& g, const Bufs& b, int parity, int bonded, int advance, hipStream_t s,
                          hipEvent_t ev_sorted) {
    // the sort passes stride over the particles with at most 2048 blocks:
    // against 512 (2M-bead melt, binning and sort per step) 62.0 -> 56.4 us,
    // and one block per 256 particles 59.2 us
    const int gs = grid_for(g.n, 2048);
    if (g.n <= kSmallSort && g.ncell <= kSmallCells) {
        hipLaunchKernelGGL(k_sort_small, dim3(1), dim3(kSmallBlock), 0, s, g, b, parity, bonded, advance);
    } else {
    hipLaunchKernelGGL(k_bin, dim3(gs), dim3(kBlock), 0, s, g, b, parity, advance);
    hipLaunchKernelGGL(k_scan_chunks, dim3(kScanBlocks), dim3(kBlock), 0, s, g, b, parity);
    hipLaunchKernelGGL(k_scatter, dim3(gs), dim3(kBlock), 0, s, g, b, parity);
    hipLaunchKernelGGL(k_rank, dim3(gs), dim3(kBlock), 0, s, g, b, parity, bonded);
    }
    if (ev_sorted) (void)hipEventRecord(ev_sorted, s);
    const int64_t nt = (g.n + kTile - 1) / kTile;
    const dim3 tiles((unsigned)(nt < kNlGrid ? nt : kNlGrid));
    const int build = list_build(g);
    if (build == MD_NL_BUILD_WAVE)
        hipLaunchKernelGGL(k_nl_wave, dim3((unsigned)((g.n + kBlock / 64 - 1) / (kBlock / 64))), dim3(kBlock), 0, s, g, b,
                           parity, bonded);
    else if (build == MD_NL_BUILD_TILES && g.le)
        hipLaunchKernelGGL(k_nl_mtile<true>, tiles, dim3(kTile), 0, s, g, b, parity, bonded);
    else if (build == MD_NL_BUILD_TILES)
        hipLaunchKernelGGL(k_nl_mtile<false>, tiles, dim3(kTile), 0, s, g, b, parity, bonded);
    else if (g.le)
        hipLaunchKernelGGL(k_nl_build_le, dim3(grid_for(g.n, 1 << 20)), dim3(kBlock), 0, s, g, b, parity, bonded);
    else
        hipLaunchKernelGGL(k_nl_build, dim3(grid_for(g.n, 1 << 20)), dim3(kBlock), 0, s, g, b, parity, bonded);
    return hipGetLastError();
}

int step_launch_grid(int64_t n, int block) {
    const int64_t t = (n + block - 1) / block;
    return (int)(t < 1 ? 1 : t);
}

template <bool BONDED, bool TENSOR>
static void launch_fast(const StepArgs& a, int block, hipStream_t s) {
    const dim3 grid((unsigned)(step_launch_grid(a.g.n, block) + a.fin)), blk((unsigned)block);
#define MD_LF(BS)                                                                                  \
    do {                                                                                           \
        if (BONDED) hipLaunchKernelGGL((k_step_fast_bonded<TENSOR, BS>), grid, blk, 0, s, a);     \
        else hipLaunchKernelGGL((k_step_fast<TENSOR, BS>), grid, blk, 0, s, a);                   \
    } while (0)
    switch (block) {
        case 64: MD_LF(64); break;
        case 128: MD_LF(128); break;
        case 512: MD_LF(512); break;
        default: MD_LF(256); break;
    }
#undef MD_LF
}

// Velocity snapshot for the DPD pair term into b.vt (the sort's scratch,
// free after the rebuild stage): (vx, vy, vz, id bits) per particle, FP32.
__global__ void __launch_bounds__(kBlock) k_snapshot_v(const Bufs b, int64_t n) {
    float4* __restrict__ out = reinterpret_cast<float4*>(b.vt);
    for (int64_t k = gtid(); k < n; k += gstride())
        out[k] = make_float4((float)b.v[k], (float)b.v[n + k], (float)b.v[2 * n + k], __uint_as_float((uint32_t)b.tag[k]));
}

hipError_t launch_step(const StepArgs& a, int fp64, int single_type, int bonded, int block, hipStream_t s) {
    const dim3 grid((unsigned)(step_launch_grid(a.g.n, block) + a.fin)), blk((unsigned)block);
    const bool w64 = block == 64;
    if (a.dy.gen && a.dy.dpd && a.mode == MODE_STEP)
        hipLaunchKernelGGL(k_snapshot_v, dim3(grid_for(a.g.n)), dim3(kBlock), 0, s, a.b, a.g.n);
    const size_t adress_tabs = 2 * sizeof(float2) * (size_t)a.g.table_points;
    const size_t pair_tab = a.pt.tabn[0] > 1 ? sizeof(float2) * (size_t)a.pt.tabn[0] : 0;
    if (a.dy.gen && a.dy.dpd && a.mode == MODE_STEP && single_type && !a.dy.adress && pair_tab <= 16384) {
        // the queue and the pair table in LDS
#define MD_LD(BO, LE)                                                                                     \
    do {                                                                                                  \
        if (w64) hipLaunchKernelGGL((k_step_dpd<BO, LE, 64>), grid, blk, pair_tab, s, a);                 \
        else hipLaunchKernelGGL((k_step_dpd<BO, LE, kBlock>), grid, blk, pair_tab, s, a);                 \
    } while (0)
        if (bonded) { if (a.g.le) MD_LD(true, true); else MD_LD(true, false); }
        else { if (a.g.le) MD_LD(false, true); else MD_LD(false, false); }
#undef MD_LD
    } else if (a.dy.gen && a.dy.adress && !a.dy.dpd && !a.g.le && single_type && a.b.tab && adress_tabs <= 32768) {
        // both tables in LDS
#define MD_LA(BO)                                                                                          \
    do {                                                                                                   \
        if (w64) hipLaunchKernelGGL((k_step_adress<BO, 64>), grid, blk, adress_tabs, s, a);                \
        else hipLaunchKernelGGL((k_step_adress<BO, kBlock>), grid, blk, adress_tabs, s, a);                \
    } while (0)
        if (bonded) MD_LA(true); else MD_LA(false);
#undef MD_LA
    } else if (a.dy.gen) {
        // tables in LDS for one particle type, when both rows fit in 32 KB
        const size_t tab_lds = 2 * sizeof(float2) * (size_t)a.g.table_points;
        const bool lds = single_type && a.b.tab && a.g.table_points >= 2 && tab_lds <= 32768;
#define MD_LG(B, S, T)                                                                                     \
    do {                                                                                                   \
        if (w64) hipLaunchKernelGGL((k_step_gen<B, S, T, 64>), grid, blk, T ? tab_lds : 0, s, a);          \
        else hipLaunchKernelGGL((k_step_gen<B, S, T, kBlock>), grid, blk, T ? tab_lds : 0, s, a);          \
    } while (0)
        if (bonded) {
            if (lds) MD_LG(true, true, true);
            else if (single_type) MD_LG(true, true, false);
            else MD_LG(true, false, false);
        } else {
            if (lds) MD_LG(false, true, true);
            else if (single_type) MD_LG(false, true, false);
            else MD_LG(false, false, false);
        }
#undef MD_LG
    } else if (fp64) {
#define MD_L64(S, B)                                                                  \
    do {                                                                              \
        if (w64) hipLaunchKernelGGL((k_step64<S, B, 64>), grid, blk, 0, s, a);        \
        else hipLaunchKernelGGL((k_step64<S, B, kBlock>), grid, blk, 0, s, a);        \
    } while (0)
        if (single_type) { if (bonded) MD_L64(true, true); else MD_L64(true, false); }
        else { if (bonded) MD_L64(false, true); else MD_L64(false, false); }
#undef MD_L64
    } else if (a.use_fast) {
        const bool t = a.tensor != 0;
        if (bonded) {
            if (t) launch_fast<true, true>(a, block, s);
            else launch_fast<true, false>(a, block, s);
        } else {
            if (t) launch_fast<false, true>(a, block, s);
            else launch_fast<false, false>(a, block, s);
        }
    } else {
#define MD_LQ(S, B, T)                                                                   \
    do {                                                                                 \
        if (w64) hipLaunchKernelGGL((k_step_q<S, B, T, 64>), grid, blk, 0, s, a);        \
        else hipLaunchKernelGGL((k_step_q<S, B, T, kBlock>), grid, blk, 0, s, a);        \
    } while (0)
        const bool t = a.tensor != 0;
        if (single_type) {
            if (bonded) { if (t) MD_LQ(true, true, true); else MD_LQ(true, true, false); }
            else { if (t) MD_LQ(true, false, true); else MD_LQ(true, false, false); }
        } else {
            if (bonded) { if (t) MD_LQ(false, true, true); else MD_LQ(false, true, false); }
            else { if (t) MD_LQ(false, false, true); else MD_LQ(false, false, false); }
        }
#undef MD_LQ
    }
    return hipGetLastError();
}

hipError_t launch_finalize(const Bufs& b, int parity, int nblocks, int block, int mode, const double* spart,
                           int tensor, hipStream_t s) {
#define MD_FIN(BS, NA) \
    hipLaunchKernelGGL((k_finalize<BS, NA>), dim3(1), dim3(BS), 0, s, b, parity, nblocks, mode, spart)
    if (tensor) MD_FIN(kFinal, kNacc);
    else if (block == 64) MD_FIN(64, kNaccStep);
    else if (block == 128) MD_FIN(128, kNaccStep);
    else if (block == 512) MD_FIN(512, kNaccStep);
    else MD_FIN(kBlock, kNaccStep);
#undef MD_FIN
    return hipGetLastError();
}

hipError_t launch_sur_step(const StepArgs& a, const SurBufs& sb, const SurConst& c, int bonded, int a_bf16,
                           hipStream_t s) {
    dim3 grid((unsigned)(step_grid(a.g.n) + a.fin)), blk(kBlock);
    const bool t = a.tensor != 0;
#define MD_LS(BO, T, A) hipLaunchKernelGGL((k_sur_step<BO, T, A>), grid, blk, 0, s, a, sb, c)
    if (a_bf16) {
        if (bonded) { if (t) MD_LS(true, true, true); else MD_LS(true, false, true); }
        else { if (t) MD_LS(false, true, true); else MD_LS(false, false, true); }
    } else {
        if (bonded) { if (t) MD_LS(true, true, false); else MD_LS(true, false, false); }
        else { if (t) MD_LS(false, true, false); else MD_LS(false, false, false); }
    }
#undef MD_LS
    return hipGetLastError();
}

}  // namespace md

namespace md {

hipError_t launch_batch_rebuild(const BatchCells& bc, const SysEntry* tab, const int32_t* tile_sys, int64_t ntiles,
                                int parity, int advance, hipStream_t s, hipEvent_t ev_sorted) {
    const dim3 tg((unsigned)ntiles), blk(kBlock);
    hipLaunchKernelGGL(k_batch_any, dim3(1), dim3(256), 0, s, bc, parity, advance);
    hipLaunchKernelGGL(k_batch_bin, tg, blk, 0, s, tab, tile_sys, parity);
    hipLaunchKernelGGL(k_scan_reduce, dim3(kScanBlocks), dim3(kBlock), 0, s, bc.gg, bc.gb);
    hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(kScanBlocks), 0, s, bc.gb);
    hipLaunchKernelGGL(k_scan_apply, dim3(kScanBlocks), dim3(kBlock), 0, s, bc.gg, bc.gb);
    hipLaunchKernelGGL(k_batch_bases, dim3(1), dim3(256), 0, s, bc);
    hipLaunchKernelGGL(k_batch_localize, dim3(grid_for(bc.gg.ncell, 4096)), blk, 0, s, bc, parity);
    hipLaunchKernelGGL(k_batch_scatter, tg, blk, 0, s, tab, tile_sys, parity);
    hipLaunchKernelGGL(k_batch_rank, tg, blk, 0, s, tab, tile_sys, parity);
    if (ev_sorted) (void)hipEventRecord(ev_sorted, s);
    hipLaunchKernelGGL(k_batch_nl, dim3((unsigned)ntiles * (kBlock / kTile)), dim3(kTile), 0, s, tab, tile_sys, parity);
    return hipGetLastError();
}

hipError_t launch_batch_step(const SysEntry* tab, const int32_t* tile_sys, int64_t ntiles, int tensor, hipStream_t s) {
    const dim3 grid((unsigned)ntiles);
    if (tensor) hipLaunchKernelGGL(k_batch_step<true>, grid, dim3(kBlock), 0, s, tab, tile_sys);
    else hipLaunchKernelGGL(k_batch_step<false>, grid, dim3(kBlock), 0, s, tab, tile_sys);
    return hipGetLastError();
}

hipError_t launch_batch_observe(const SysEntry* tab, int nsys, hipStream_t s) {
    hipLaunchKernelGGL(k_batch_observe, dim3(nsys), dim3(kFinal), 0, s, tab);
    return hipGetLastError();
}

hipError_t launch_batch_end(const BatchCells& bc, hipStream_t s) {
    hipLaunchKernelGGL(k_batch_end, dim3(1), dim3(256), 0, s, bc);
    return hipGetLastError();
}

hipError_t launch_batch_gather_obs(const SysEntry* tab, int nsys, double* out, hipStream_t s) {
    hipLaunchKernelGGL(k_batch_gather_obs, dim3(1), dim3(256), 0, s, tab, nsys, out);
    return hipGetLastError();
}

}  // namespace md
