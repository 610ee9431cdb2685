// sr_pic.hip -- closing the PIC loop around the emission step: the Yee field
// solve, the grid charge and the charge-conserving current of the particles'
// moves, and the ballistic motion of the emitted photons.
//
// The paper's emission method runs inside a PIC code: particles on a grid,
// Maxwell's equations for the field, the particles' currents feeding it
// (section "The field setup"); the photons it emits are particles that move at
// c along their direction.  Normalised units: E, B in m c omega_r / e, lengths
// in c/omega_r, densities in n_r = m omega_r^2 / (4 pi e^2), so
//     dB/dt = -curl E,   dE/dt = curl B - J,   div E = rho.
// A step keeps E and B at whole steps, where the particles gather them:
//     B -= (dt/2) curl E;   E += dt (curl B - J);   B -= (dt/2) curl E.
#include <math.h>

#include <type_traits>

#include "sr_common.hpp"

namespace sr {
namespace {

// Grid geometry for the PIC kernels (positions from the lower corner).
struct PicGrid {
    int n[3];
    float inv_hi[3], inv_lo[3];   // 1/dx split so that x/dx keeps ~2^-24 absolute accuracy
    float L[3];                   // box lengths
    float dV;                     // cell volume (2D: dx dy)
};

inline int pic_grid(const sr_grid *g, PicGrid &G) {
    if (!g || (g->dim != 2 && g->dim != 3)) return SR_E_INVAL;
    if (g->dim == 2 && g->n[2] != 1) return SR_E_INVAL;
    int64_t cells = 1;
    for (int a = 0; a < 3; ++a) {
        if (g->n[a] < 1 || g->n[a] > (1 << 24)) return SR_E_INVAL;
        if (a < g->dim && (!(g->dx[a] > 0.0) || !isfinite(g->dx[a]))) return SR_E_INVAL;
        cells *= g->n[a];
    }
    if (cells >= (int64_t)1 << 30) return SR_E_UNSUPPORTED;
    G.dV = 1.0f;
    for (int a = 0; a < 3; ++a) {
        G.n[a] = (int)g->n[a];
        const double inv = a < g->dim ? 1.0 / g->dx[a] : 0.0;
        G.inv_hi[a] = (float)inv;
        G.inv_lo[a] = (float)(inv - (double)G.inv_hi[a]);
        G.L[a] = a < g->dim ? (float)(g->n[a] * g->dx[a]) : 0.0f;
        if (a < g->dim) G.dV *= (float)g->dx[a];
    }
    return SR_OK;
}

__device__ __forceinline__ uint32_t cell(int i, int j, int k, const PicGrid &G) {
    return (uint32_t)i + (uint32_t)G.n[0] * ((uint32_t)j + (uint32_t)G.n[1] * (uint32_t)k);
}
__device__ __forceinline__ int up(int i, int n) { return i + 1 == n ? 0 : i + 1; }
__device__ __forceinline__ int dn(int i, int n) { return i == 0 ? n - 1 : i - 1; }

// ------------------------------------------------------------ Yee field solve
// B -= h curl E on the B points (forward differences), one thread per cell.
template <int DIM>
__global__ __launch_bounds__(256) void curl_e_kernel(const float *__restrict__ ex,
                                                     const float *__restrict__ ey,
                                                     const float *__restrict__ ez,
                                                     float *__restrict__ bx, float *__restrict__ by,
                                                     float *__restrict__ bz, PicGrid G, float hx,
                                                     float hy, float hz, uint32_t cells) {
    const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= cells) return;
    const int nx = G.n[0], ny = G.n[1];
    const int i = (int)(c % (uint32_t)nx), r = (int)(c / (uint32_t)nx);
    const int j = r % ny, k = r / ny;
    const uint32_t cx = cell(up(i, nx), j, k, G), cy = cell(i, up(j, ny), k, G);
    const float ex0 = ld(ex, c), ey0 = ld(ey, c), ez0 = ld(ez, c);
    // hx = h/dx etc.
    float dbx = hy * (ld(ez, cy) - ez0);
    float dby = -hx * (ld(ez, cx) - ez0);
    const float dbz = hx * (ld(ey, cx) - ey0) - hy * (ld(ex, cy) - ex0);
    if (DIM == 3) {
        const uint32_t cz = cell(i, j, up(k, G.n[2]), G);
        dbx -= hz * (ld(ey, cz) - ey0);
        dby += hz * (ld(ex, cz) - ex0);
    }
    st(bx, c, ld(bx, c) - dbx);
    st(by, c, ld(by, c) - dby);
    st(bz, c, ld(bz, c) - dbz);
}

// E += dt (curl B - J) on the E points (backward differences).
template <int DIM, bool HAS_J>
__global__ __launch_bounds__(256) void curl_b_kernel(float *__restrict__ ex, float *__restrict__ ey,
                                                     float *__restrict__ ez,
                                                     const float *__restrict__ bx,
                                                     const float *__restrict__ by,
                                                     const float *__restrict__ bz,
                                                     const float *__restrict__ jx,
                                                     const float *__restrict__ jy,
                                                     const float *__restrict__ jz, PicGrid G,
                                                     float dt, float tx, float ty, float tz,
                                                     uint32_t cells) {
    const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= cells) return;
    const int nx = G.n[0], ny = G.n[1];
    const int i = (int)(c % (uint32_t)nx), r = (int)(c / (uint32_t)nx);
    const int j = r % ny, k = r / ny;
    const uint32_t cx = cell(dn(i, nx), j, k, G), cy = cell(i, dn(j, ny), k, G);
    const float bx0 = ld(bx, c), by0 = ld(by, c), bz0 = ld(bz, c);
    // tx = dt/dx etc.
    float dex = ty * (bz0 - ld(bz, cy));
    float dey = -tx * (bz0 - ld(bz, cx));
    float dez = tx * (by0 - ld(by, cx)) - ty * (bx0 - ld(bx, cy));
    if (DIM == 3) {
        const uint32_t cz = cell(i, j, dn(k, G.n[2]), G);
        dex -= tz * (by0 - ld(by, cz));
        dey += tz * (bx0 - ld(bx, cz));
    }
    if (HAS_J) {
        dex = fmaf(-dt, ld(jx, c), dex);
        dey = fmaf(-dt, ld(jy, c), dey);
        dez = fmaf(-dt, ld(jz, c), dez);
    }
    st(ex, c, ld(ex, c) + dex);
    st(ey, c, ld(ey, c) + dey);
    st(ez, c, ld(ez, c) + dez);
}

// --------------------------------------------------- charge and current
// Position on one axis as (cell index, fraction in [0, 1)).
__device__ __forceinline__ void locate(float x, float inv_hi, float inv_lo, int n, int &i, float &f) {
    const float u = x * inv_hi;
    float fi = floorf(u);
    float fr = fmaf(x, inv_hi, -fi) + x * inv_lo;
    if (fr < 0.0f) { fr += 1.0f; fi -= 1.0f; }
    if (fr >= 1.0f) { fr -= 1.0f; fi += 1.0f; }
    i = (int)fi;
    i = i < 0 ? i + n : (i >= n ? i - n : i);
    i = min(max(i, 0), n - 1);
    f = fr;
}

// Node index base + c (c = 0..3, base = i - 1) wrapped into [0, n).
__device__ __forceinline__ int node(int i, int c, int n) {
    int v = i - 1 + c;
    v = v < 0 ? v + n : (v >= n ? v - n : v);
    return min(max(v, 0), n - 1);
}

// l / d for 0 <= l < 2^22 and d >= 1, from a float reciprocal: the product
// is within one of the quotient, and one step each way corrects it
__device__ __forceinline__ int div_small(int l, int d, float inv_d) {
    int q = (int)((float)l * inv_d);
    q -= q * d > l ? 1 : 0;
    q += (q + 1) * d <= l ? 1 : 0;
    return q;
}

// i in [-2n, 3n) onto [0, n)
__device__ __forceinline__ int wrap2(int i, int n) {
    if (i < 0) i += n;
    if (i < 0) i += n;
    if (i >= n) i -= n;
    if (i >= n) i -= n;
    return i;
}

// CIC weight of a particle at relative coordinate r (cells from node i) on the
// node i - 1 + c.
__device__ __forceinline__ float cic_w(float r, int c) {
    return fmaxf(0.0f, 1.0f - fabsf(r - (float)(c - 1)));
}

// A cell unwrapped across the periodic boundary to the copy nearest the block's first
// particle's.
__device__ __forceinline__ int unwrap_cell(int i, int ref, int n) {
    int d = i - ref;
    if (2 * d > n) d -= n;
    else if (2 * d < -n) d += n;
    return ref + d;
}

// A deposit block first finds the box of nodes its particles touch, with cells
// taken relative to the block's first particle across the periodic boundary (a
// block whose sorted particles run from the end of one tile row into the next
// keeps a compact box).  A box above `cap` nodes (particles that have drifted
// far since the last sort) is taken in up to kDepSlabs slabs along its widest axis,
// each particle in the slab of its cell, with the LDS of one: that costs the slabs'
// common nodes twice, where a particle outside the box adds to the grid by itself.
// Slabs are taken one after another, so a launch whose blocks do not fill the chip is
// allowed fewer (max_slabs).  A box too large for its slabs (an unsorted ensemble) is
// none (false), or with WINDOW shrinks, widest axis first, to a window of at most `cap`
// nodes about the block's mean cell; the particles whose nodes leave the window add to
// the grid directly.
struct DepShared {
    int ref[3], lo[3], hi[3];   // first particle's cell; smallest and largest unwrapped cells
    uint32_t bmax;              // largest bound, as bits (no bound is negative)
    float sum[3];               // window only: sums of the cells relative to ref
    int cnt;
};
struct DepBox {
    int org[3], ext[3];   // first node (unwrapped) and extent on each axis
    float bnd;            // the block's largest bound (infinite if one is not finite)
    int slabs, axis, per; // slabs of `per` cells along `axis`
};
constexpr int kDepSlabs = 8;        // at most

// Slab t of the box (the box itself if there is one): its own box, and whether it is
// the slab of the cell U.
template <int DIM>
__device__ __forceinline__ bool deposit_slab(const DepBox &bx, int t, int below, int above,
                                             const int U[3], DepBox &w) {
    w = bx;
    if (bx.slabs == 1) return true;
    bool mine = false;
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        if (a != bx.axis) continue;
        const int first = t * bx.per, c = U[a] - (bx.org[a] + below) - first;
        w.org[a] = bx.org[a] + first;
        w.ext[a] = min(bx.per, bx.ext[a] - below - above - first) + below + above;
        mine = c >= 0 && c < bx.per;
    }
    return mine;
}

// The box of the block's live particles: I their cells, `bound` >= 0 a bound on
// each one's contributions; nodes reach from `below` under the smallest cell to
// `above` over the largest.  U receives the particle's unwrapped cell.  False
// when no particle is live, or without a box.  Call with the whole block (thread 0
// active).
template <int DIM, bool WINDOW>
__device__ __forceinline__ bool deposit_box(DepShared &sh, const int I[3], bool live, float bound,
                                            const PicGrid &G, int below, int above, int cap,
                                            int max_slabs, int U[3], DepBox &bx) {
    if (threadIdx.x == 0) {
        for (int a = 0; a < 3; ++a) {
            sh.ref[a] = I[a];
            sh.lo[a] = 0x3fffffff;
            sh.hi[a] = -0x3fffffff;
            sh.sum[a] = 0.0f;
        }
        sh.bmax = 0;
        sh.cnt = 0;
    }
    __syncthreads();
#pragma unroll
    for (int a = 0; a < 3; ++a) U[a] = a < DIM ? unwrap_cell(I[a], sh.ref[a], G.n[a]) : I[a];
    const int lane = threadIdx.x & 63;
    // wave reductions, then one LDS atomic a wave: every thread reads one value each
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        const int lo = wave_min_i(live ? U[a] : 0x3fffffff);
        const int hi = wave_max_i(live ? U[a] : -0x3fffffff);
        if (lane == 0) {
            atomicMin(&sh.lo[a], lo);
            atomicMax(&sh.hi[a], hi);
        }
    }
    {
        const float b = wave_max(live ? (bound <= 3.0e38f ? bound : __builtin_inff()) : 0.0f);
        if (lane == 0) atomicMax(&sh.bmax, __float_as_uint(b));
    }
    __syncthreads();
    bool any = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        bx.org[a] = 0;
        bx.ext[a] = 1;
        if (a >= DIM) continue;
        const int lo = sh.lo[a], hi = sh.hi[a];
        any = any && hi >= lo;      // no live particle: lo > hi
        bx.org[a] = lo - below;
        bx.ext[a] = hi - lo + below + above + 1;
    }
    bx.bnd = __uint_as_float(sh.bmax);
    if (!any) return false;
    bx.slabs = 1;
    bx.axis = 0;
    bx.per = 0;
    // volumes in 64 bits: extents can be as large as the grid
    int64_t vol = (int64_t)bx.ext[0] * bx.ext[1] * bx.ext[2];
    if (vol <= cap) return true;
    {
        int wide = 0, len = bx.ext[0], area = 1;      // the widest axis, and the section across it
#pragma unroll
        for (int b = 1; b < DIM; ++b)
            if (bx.ext[b] > len) { wide = b; len = bx.ext[b]; }
#pragma unroll
        for (int b = 0; b < DIM; ++b)
            if (b != wide) area = min(area * min(bx.ext[b], cap + 1), cap + 1);
        const int per = cap / area - below - above;
        const int n_cells = len - below - above;
        if (per >= 1 && n_cells <= max_slabs * per) {
            bx.axis = wide;
            bx.slabs = (n_cells + per - 1) / per;
            bx.per = (n_cells + bx.slabs - 1) / bx.slabs;   // even slabs,
            bx.slabs = (n_cells + bx.per - 1) / bx.per;     // none of them empty
            return true;
        }
    }
    if (!WINDOW) return false;
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        const float v = wave_sum_f(live ? (float)(U[a] - sh.ref[a]) : 0.0f);
        if (lane == 0) atomicAdd(&sh.sum[a], v);
    }
    const int n_live = (int)__popcll(__ballot(live));
    if (lane == 0) atomicAdd(&sh.cnt, n_live);
    __syncthreads();
    const int cnt = sh.cnt;
    for (int it = 0; it < DIM && vol > cap; ++it) {
        int wide = 0;
#pragma unroll
        for (int b = 1; b < DIM; ++b)
            if (bx.ext[b] > (wide == 0 ? bx.ext[0] : bx.ext[1])) wide = b;
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
            if (a != wide) continue;
            const int64_t other = vol / bx.ext[a];
            const int wdt = (int)min<int64_t>(bx.ext[a], max<int64_t>(4, cap / other));
            const int c = sh.ref[a] + (int)floorf(sh.sum[a] / (float)max(cnt, 1) + 0.5f);
            bx.org[a] = min(max(c - wdt / 2, bx.org[a]), bx.org[a] + bx.ext[a] - wdt);
            bx.ext[a] = wdt;
            vol = other * wdt;
        }
    }
    return true;
}

// The grid index of the first node of each row (y, z) of the box, wrapped onto the
// periodic grid: the nodes lie in [-n/2 - 1, 3n/2 + 1], so two wraps each way reach
// [0, n) for any n.  Call with the whole block, and synchronise after it.
template <int DIM>
__device__ __forceinline__ void box_rows(uint32_t *row, const DepBox &bx, const PicGrid &G) {
    const float inv_e1 = 1.0f / (float)bx.ext[1];
    for (int r = threadIdx.x; r < bx.ext[1] * bx.ext[2]; r += blockDim.x) {
        const int lk = div_small(r, bx.ext[1], inv_e1), lj = r - lk * bx.ext[1];
        int j = wrap2(bx.org[1] + lj, G.n[1]), k = DIM == 3 ? wrap2(bx.org[2] + lk, G.n[2]) : 0;
        j = min(max(j, 0), G.n[1] - 1);
        k = min(max(k, 0), G.n[2] - 1);
        row[r] = cell(0, j, k, G);
    }
}
// Grid index of box node l (x fastest).
__device__ __forceinline__ uint32_t box_node(int l, const uint32_t *row, const DepBox &bx, float inv_e0,
                                             const PicGrid &G) {
    const int r = div_small(l, bx.ext[0], inv_e0);
    const int i = wrap2(bx.org[0] + l - r * bx.ext[0], G.n[0]);
    return row[r] + (uint32_t)min(max(i, 0), G.n[0] - 1);
}

// Charge: rho += q w S / dV on the 4 (2D) or 8 (3D) nodes of each particle.
//
// Added one by one, the contributions of sorted particles are scattered float
// atomics of one lane each, which is what the deposit took its time for.  The
// block sums them in its LDS box instead and adds the box's nodes to the grid,
// consecutive lanes on consecutive nodes.  The sums are exact: a contribution
// v, the same binary32 product as on the direct path, becomes the integer
// v 2^(kRhoBits - e) with 2^e above the block's largest |q w / dV|, rounded at
// 2^(e - kRhoBits - 1); a particle lighter than 2^-18 of the heaviest, where
// that could lose bits a float would keep, and one whose weight or position is
// not finite, adds to the grid directly.  At most 2^8 contributions of at most
// 2^44 units meet on a node, so a sum stays below 2^53 and its conversion back
// is exact too: a node's block sum is rounded once.  A block without a box (an
// unsorted ensemble) goes direct.
//
// The sort and the deposit of 4.0 M electrons at 1/4 per cell on 256^3 take 264 us
// where the direct adds took 900.  At that density a block's box is 6 nodes a particle
// whatever its size, so small blocks win as long as a block that straddles two tile
// rows keeps to one or two slabs: 292 us with 128 particles and 2048 nodes, 333 with 512
// and 6144, 497 with 1024 and 7936.  With 256 the blocks in flight decide: five a
// compute unit with 3072 nodes; 266 and 268 us with four and 3840 or 3584, 285 with
// 4096 nodes and the 88 registers the compiler takes by itself.
constexpr int kRhoThreads = 256;   // particles per block
constexpr int kRhoCells = 3072;    // 24 KB and 6 KB of rows: five blocks per compute unit
constexpr int kRhoBits = 44;

// v 2^s as a 64-bit integer, for |v 2^s| < 2^51: the sum with 1.5 2^52 leaves
// the integer, in two's complement, in the low bits of the significand
__device__ __forceinline__ unsigned long long fixed64(float v, double scale) {
    const double b = fma((double)v, scale, 6755399441055744.0);
    return (unsigned long long)(__double_as_longlong(b) - 0x4338000000000000ll);
}

// A particle's charge on its nodes, as add(offsets a, b, c in 0..1 from its cell, value).
template <int DIM, typename ADD>
__device__ __forceinline__ void charge_each(const float F[3], float qw, ADD &&add) {
#pragma unroll
    for (int c = 0; c < (DIM == 3 ? 2 : 1); ++c)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                const float wt = (a ? F[0] : 1.0f - F[0]) * (b ? F[1] : 1.0f - F[1]) *
                                 (DIM == 3 ? (c ? F[2] : 1.0f - F[2]) : 1.0f);
                add(a, b, c, qw * wt);
            }
}
template <int DIM>
__device__ __forceinline__ void charge_direct(const int I[3], const float F[3], float qw, const PicGrid &G,
                                              float *__restrict__ rho) {
    charge_each<DIM>(F, qw, [&](int a, int b, int c, float v) {
        const int i = node(I[0], 1 + a, G.n[0]), j = node(I[1], 1 + b, G.n[1]);
        const int k = DIM == 3 ? node(I[2], 1 + c, G.n[2]) : 0;
        unsafeAtomicAdd(&rho[cell(i, j, k, G)], v);
    });
}

// The direct adds alone, for what the box does not pay for: a box block is a chain of
// some 3 us and 2 us a slab, and where few particles share a node it adds as often.
// Box against direct, us, right after the sort and one cell of drift later: 3D 12 000
// electrons at 2 per cell 6.5 and 6.3 against 6.4 and 6.2; 40 000 at 1/4 10 and 14 against 12
// and 14, at 0.06 14 and 19 against 13 and 15; 80 000 at 0.06 17 and 28 against 25 and 29; 2D
// 80 000 at 1/2 7.6 and 8.3 against 9.2 and 10.1, at 0.06 14 and 21 against 13 and 14.
// From 2^21 adds on a box is sought at any density (a set can be dense in a thin part of
// its grid): 300 000 unsorted 120 against 118 us, sorted at 0.03 56 against 98.  Eight
// slabs at that size: 1 M at 0.06 in 2D 68 us, 91 with up to two; below it four: 80 000 in
// 3D at 1/2 three cells of drift after the sort 34 us, 43 with up to eight.
constexpr int64_t kRhoAnyAdds = (int64_t)1 << 21, kRhoMinAdds = (int64_t)1 << 18;
constexpr double kRhoMinShared = 40960.0;      // n adds / cells
inline int rho_slabs(int64_t n, int dim, double cells) {      // 0: direct
    const int64_t adds = n << dim;
    if (adds >= kRhoAnyAdds) return kDepSlabs;
    return adds >= kRhoMinAdds && (double)n * (double)adds >= kRhoMinShared * cells ? 4 : 0;
}
template <int DIM>
__global__ __launch_bounds__(kRhoThreads) void rho_direct_kernel(sr_particles_f32 P, PicGrid G, float qv,
                                                                 float *__restrict__ rho) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= P.n) return;
    const uint32_t u = (uint32_t)p;
    int I[3] = {0, 0, 0};
    float F[3] = {0.0f, 0.0f, 0.0f};
    for (int a = 0; a < DIM; ++a) locate(ld(P.x[a], u), G.inv_hi[a], G.inv_lo[a], G.n[a], I[a], F[a]);
    charge_direct<DIM>(I, F, qv * ld(P.w, u) / G.dV, G, rho);
}

template <int DIM>
__global__ __launch_bounds__(kRhoThreads) __attribute__((amdgpu_waves_per_eu(5))) void rho_kernel(sr_particles_f32 P, PicGrid G, float qv,
                                                          float *__restrict__ rho, int max_slabs) {
    __shared__ unsigned long long box[kRhoCells];
    __shared__ uint32_t row[kRhoCells / 2];      // a box is at least 2 nodes wide
    __shared__ DepShared sh;
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool active = p < P.n;
    const uint32_t u = active ? (uint32_t)p : 0u;
    int I[3] = {0, 0, 0};
    float F[3] = {0.0f, 0.0f, 0.0f};
    for (int a = 0; a < DIM; ++a) locate(ld(P.x[a], u), G.inv_hi[a], G.inv_lo[a], G.n[a], I[a], F[a]);
    const float qw = qv * ld(P.w, u) / G.dV;
    bool fin = fabsf(qw) <= 3.0e38f;
    for (int a = 0; a < DIM; ++a) fin = fin && fabsf(F[a]) <= 1.0f;
    const bool live = active && fin && qw != 0.0f;
    int U[3];
    DepBox bx;
    const bool boxed =
        deposit_box<DIM, false>(sh, I, live, fabsf(qw), G, 0, 1, kRhoCells, max_slabs, U, bx);
    const bool in_box = live && boxed && fabsf(qw) * 262144.0f >= bx.bnd;
    if (active && !in_box && (qw != 0.0f || !fin))
        charge_direct<DIM>(I, F, qw, G, rho);
    if (!boxed) return;            // the condition is block-wide
    __syncthreads();               // (not for the data: 263 us for the sort and deposit, 266 without)
    int e = 0;
    (void)frexpf(bx.bnd, &e);      // bnd < 2^e
    const double to_fix = ldexp(1.0, kRhoBits - e), from_fix = ldexp(1.0, e - kRhoBits);
    for (int t = 0; t < bx.slabs; ++t) {
        DepBox w;
        const bool mine = deposit_slab<DIM>(bx, t, 0, 1, U, w) && in_box;
        const int cells = w.ext[0] * w.ext[1] * w.ext[2];
        if (t) __syncthreads();        // the box is flushed
        for (int q = threadIdx.x; q < cells; q += kRhoThreads) box[q] = 0;
        box_rows<DIM>(row, w, G);
        __syncthreads();
        if (mine) {
            const int l0 = (U[0] - w.org[0]) +
                           w.ext[0] * ((U[1] - w.org[1]) + w.ext[1] * (DIM == 3 ? U[2] - w.org[2] : 0));
            charge_each<DIM>(F, qw, [&](int a, int b, int c, float v) {
                atomicAdd(&box[l0 + a + w.ext[0] * (b + w.ext[1] * c)], fixed64(v, to_fix));
            });
        }
        __syncthreads();
        const float inv_e0 = 1.0f / (float)w.ext[0];
        for (int q = threadIdx.x; q < cells; q += kRhoThreads) {
            const long long sum = (long long)box[q];
            if (sum != 0)
                unsafeAtomicAdd(&rho[box_node(q, row, w, inv_e0, G)], (float)((double)sum * from_fix));
        }
    }
}

// Esirkepov's current of the move x_old -> x (one lane per particle).  On each
// axis the old shape S0 and the new shape S1 of a move below one cell lie on
// three consecutive nodes among i-1 .. i+2 of the old cell i; D = S1 - S0.  Per node
// of the stencil
//   3D  W_x = Dx (S0y S0z + Dy S0z/2 + S0y Dz/2 + Dy Dz/3)  (and cyclically),
//   Jx(i+1/2) = Jx(i-1/2) - q w (dx/dt) W_x / dV, summed along x;
//   2D  W_x = Dx (S0y + Dy/2),  W_y = Dy (S0x + Dx/2),
//       Jz = q w v_z (S0x S0y + Dx S0y/2 + S0x Dy/2 + Dx Dy/3) / dV on the nodes.
// A move of a cell or more sets *status.
//
// Most moves stay in their cell.  Then S0 and S1 share two nodes, D = (-du, du) with
// du the move in cells, and only the first partial sum along an axis is not zero: 12
// contributions a particle in 3D, 8 in 2D, where the general stencil has 54 (3D) and,
// with some lane of nearly every wave crossing a cell face, every wave paid for them
// all.  Each block adds the moves that stay at once and lists the others, which it then
// takes densely, 64 to a wave.
//
// Sorted particles put the lanes of a block on the same few cells, where
// global float atomics serialise: the block accumulates in its LDS box
// (deposit_box, kDepCells cells, three components) and adds the box's non-zero
// entries to the grid at the end, the three components of a node together.
//
// The box holds fixed-point integers, not floats: on gfx950 an LDS float
// atomic add takes about 40 times as long as an integer one, and it was the
// bulk of the deposit's time.  Each contribution v is rounded to an integer
// multiple of 2^(e-21), where 2^e bounds every contribution of the block: on
// each axis |v| <= |c_a| |du_a| (the partial sums of D over a hat shape are
// bounded by the move du in cells, the transverse factor lies in [0, 1]), and
// |v| <= |c_z| for the 2D Jz.  A node takes at most one contribution per
// particle and component, so a sum stays below 512 * 2^21 = 2^30, and the
// integer adds are exact and independent of order.  The rounding error per
// contribution is at most half a unit, 2^(e-22) <= 2^-21 B with B the block's
// largest bound, so a node's block sum is within n 2^-21 B <= 2^-12 B of the
// exact sum of its n <= 512 contributions.  That bound is absolute: a node
// whose current is far below B in a block that also holds a much heavier or
// faster particle keeps only that absolute accuracy.
//
// The particles of a box taken in slabs would otherwise add to the grid in 32 bits, most
// of them, and lose nothing by it here: a slab's unit is 2^(e-31) with 2^e above the sum
// S of its particles' bounds, which is all that a node's sum can reach (the bounds carry a
// margin of a thousandth), and particles whose bound is below 2^-12 S add to the grid
// directly.  Against 64 bits, rms error over rms current, as so, with one window and direct
// adds, and with the units of a box taken at once: 65 536 electrons on 64^3, 0.3 cells
// after their sort, 1.2e-6, 2.1e-6, 3.5e-6; 200 000 on 300^2, ten cells after it, 1.3e-6,
// 1.9e-6, 2.1e-6.
//
// 2^23 electrons, two a cell, in 4x4x4 tiles take 310 us right after the sort, where
// the general stencil for all of them took 437; 380 us after 407 steps of a wake, 686
// before, when a drifted block's particles beyond the window went to the grid one by
// one.  Of these the blocks' set-up and loads are some 128 us and the entries' atomics
// some 50.  Bound by latency at that: six waves per SIMD (80 registers; with the 88 that
// the compiler takes by itself there are only five, and a third block does not fit).
constexpr int kDepThreads = 512;   // particles per block
constexpr int kDepCells = 3072;
constexpr int kDepRows = kDepCells / 4;   // a box is at least 4 nodes wide
// 2^kDepFracBits units per bound and at most kDepThreads contributions per
// node: sums stay below 2^30
constexpr int kDepFracBits = 30 - 9;
static_assert(kDepThreads == 512, "kDepFracBits assumes 2^9 particles per block");
constexpr int kDepSumBits = 31;           // in slabs: S lies below 2^kDepSumBits units
constexpr float kDepLight = 0x1p-12f;     // of S
// Slabs are a chain, so where the blocks do not fill the chip fewer are allowed.  Times with
// direct adds over times with up to two, four and eight slabs, sets from two electrons per
// cell to 0.003, at 0.3 to 10 cells after their sort, mean (worst): 3D 12 000 1.14 (1.04),
// 1.13 (0.93), 1.03 (0.59); 40 000 1.07, 1.09, 1.07 (1.02 all three); 200 000 1.03, 1.07,
// 1.13 (1.00).  2D 24 000 1.21 (1.08), 1.15 (0.95), 1.00 (0.62); 100 000 1.11, 1.15, 1.19
// (1.03); 140 000 1.12 (1.01), 1.13 (0.91), 1.13 (0.87); 200 000 1.10, 1.18, 1.25 (1.01).
inline int current_slabs(int64_t n, int dim) {
    if (dim == 3) return n < 24576 ? 2 : n < 40960 ? 4 : kDepSlabs;
    return n < 65536 ? 2 : n < 196608 ? 4 : kDepSlabs;
}

struct Move {
    int I[3];              // old cell of the particle on each axis
    float f0[3], du[3];    // old fraction in it, move in cells
    float cx, cy, cz;      // -q w (dx_a/dt)/dV (3D), and q w v_z / dV for 2D Jz in cz
    float bound;           // bound on |contribution| (with a margin for rounding)
    bool live;             // active, finite move below one cell
};

struct Stencil {
    int o[3];              // the move's three nodes on each axis: I - 1 + o .. I + 1 + o
    float S0[3][3], D[3][3];   // old shape and its change on those nodes
    float cx, cy, cz;
};

template <int DIM>
__device__ __forceinline__ Move make_move(const sr_particles_f32 &P, const float *const xo[3],
                                          const PicGrid &G, float qv, float inv_dt, uint32_t u,
                                          bool active, bool &bad) {
    Move s;
    s.live = active;
    bad = false;
#pragma unroll
    for (int a = 0; a < 3; ++a) { s.I[a] = 0; s.f0[a] = 0.0f; s.du[a] = 0.0f; }
    s.cx = s.cy = s.cz = 0.0f;
    s.bound = 0.0f;
    if (!active) return s;
    bool ok = true;
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        const float x0 = ld(xo[a], u), x1 = ld(P.x[a], u);
        float d = x1 - x0;                       // the shorter way round the box
        if (d > 0.5f * G.L[a]) d -= G.L[a];
        else if (d < -0.5f * G.L[a]) d += G.L[a];
        locate(x0, G.inv_hi[a], G.inv_lo[a], G.n[a], s.I[a], s.f0[a]);
        s.du[a] = d * G.inv_hi[a];
        ok = ok && fabsf(s.du[a]) < 1.0f;
    }
    if (!ok) {
        bad = true;
        s.live = false;
        return s;
    }
    const float qw = qv * ld(P.w, u);
    const float inv_dV = 1.0f / G.dV;
    s.cx = -qw * inv_dt * inv_dV / (G.inv_hi[0] + G.inv_lo[0]);
    s.cy = -qw * inv_dt * inv_dV / (G.inv_hi[1] + G.inv_lo[1]);
    if (DIM == 3) {
        s.cz = -qw * inv_dt * inv_dV / (G.inv_hi[2] + G.inv_lo[2]);
    } else {
        // v_z of the move from the momentum the position push used
        const float pz = ld(P.p[2], u), px = ld(P.p[0], u), py = ld(P.p[1], u);
        s.cz = qw * pz * __builtin_amdgcn_rsqf(1.0f + px * px + py * py + pz * pz) * inv_dV;
    }
    // |v| <= |c_a| |du_a| per axis (2D Jz: |c_z|); the margin covers the
    // rounding of the weights and of their partial sums
    constexpr float kPad = 1.0f / (1 << 20);
    float b = fmaxf(fabsf(s.cx) * (fabsf(s.du[0]) + kPad), fabsf(s.cy) * (fabsf(s.du[1]) + kPad));
    b = fmaxf(b, DIM == 3 ? fabsf(s.cz) * (fabsf(s.du[2]) + kPad) : fabsf(s.cz));
    s.bound = b * 1.001f;
    return s;
}

// The move stays in its cell on every axis.
template <int DIM>
__device__ __forceinline__ bool stays(const Move &m) {
    bool in = true;
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        const float r1 = m.f0[a] + m.du[a];
        in = in && r1 >= 0.0f && r1 < 1.0f;
    }
    return in;
}

template <int DIM>
__device__ __forceinline__ Stencil make_stencil(const Move &m) {
    Stencil s;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        s.o[a] = 1;
        for (int c = 0; c < 3; ++c) { s.S0[a][c] = (a >= DIM && c == 0) ? 1.0f : 0.0f; s.D[a][c] = 0.0f; }
    }
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        const float r1 = m.f0[a] + m.du[a];
        // old shape on nodes i, i+1; new shape on i-1, i (r1 < 0) or on
        // i, i+1 or i+1, i+2: three nodes from i - 1 + o
        const int o = r1 < 0.0f ? 0 : 1;
        s.o[a] = o;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            s.S0[a][c] = cic_w(m.f0[a], c + o);
            s.D[a][c] = cic_w(r1, c + o) - s.S0[a][c];
        }
    }
    s.cx = m.cx;
    s.cy = m.cy;
    s.cz = m.cz;
    return s;
}

// S0 S0' + D S0'/2 + S0 D'/2 + D D'/3, its roundings fixed (both stencils below are one
// arithmetic).
__device__ __forceinline__ float cross_factor(float S0, float D, float T0, float E) {
    return fmaf(D * E, 1.0f / 3.0f, fmaf(E, 0.5f * S0, fmaf(0.5f * D, T0, S0 * T0)));
}

// The contributions of a move that stays in its cell, as add(component, node offsets
// ci, cj, ck in 0..1 from cell I, value): those of the general stencil below that can be
// other than zero (but for the rounding of D), in the same arithmetic.
template <int DIM, typename ADD>
__device__ __forceinline__ void esirkepov_stay(const Move &m, ADD &&add) {
    float S0[3][2], D[3][2];
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        const float r1 = m.f0[a] + m.du[a];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            S0[a][c] = cic_w(m.f0[a], c + 1);
            D[a][c] = cic_w(r1, c + 1) - S0[a][c];
        }
    }
    const auto cross = [&](int a, int b, int i, int j) {
        return cross_factor(S0[a][i], D[a][i], S0[b][j], D[b][j]);
    };
#pragma unroll
    for (int k = 0; k < (DIM == 3 ? 2 : 1); ++k)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (DIM == 3) {
                add(0, 0, j, k, m.cx * D[0][0] * cross(1, 2, j, k));
                add(1, j, 0, k, m.cy * D[1][0] * cross(0, 2, j, k));
                add(2, j, k, 0, m.cz * D[2][0] * cross(0, 1, j, k));
            } else {
                add(0, 0, j, 0, m.cx * D[0][0] * fmaf(0.5f, D[1][j], S0[1][j]));
                add(1, j, 0, 0, m.cy * D[1][0] * fmaf(0.5f, D[0][j], S0[0][j]));
                add(2, 0, j, 0, m.cz * cross(0, 1, 0, j));
                add(2, 1, j, 0, m.cz * cross(0, 1, 1, j));
            }
        }
}

// The contributions of one particle, as add(component, node offsets ci, cj, ck in 0..2
// relative to I - 1 + o, value); with ALL those that are zero too (an add to LDS costs
// less than the test).  Along the component's own
// axis only the first two partial sums are stored: the third is the sum of D,
// which is zero.
template <int DIM, bool ALL, typename ADD>
__device__ __forceinline__ void esirkepov(const Stencil &s, ADD &&add) {
    // axis A's component on the other axes' nodes (p on axis P, q on axis Q)
    const auto along = [&](auto A, auto P, auto Q, float c) {
        constexpr int a = decltype(A)::value, pa = decltype(P)::value, qa = decltype(Q)::value;
        for (int q = 0; q < (DIM == 3 ? 3 : 1); ++q)
            for (int p = 0; p < 3; ++p) {
                const float f = DIM == 3 ? cross_factor(s.S0[pa][p], s.D[pa][p], s.S0[qa][q], s.D[qa][q])
                                         : fmaf(0.5f, s.D[pa][p], s.S0[pa][p]);
                if (!ALL && f == 0.0f) continue;
                float acc = 0.0f;
                for (int i = 0; i < 2; ++i) {
                    acc += c * s.D[a][i] * f;
                    int at[3] = {0, 0, 0};
                    at[a] = i;
                    at[pa] = p;
                    if (DIM == 3) at[qa] = q;
                    if (ALL || acc != 0.0f) add(a, at[0], at[1], at[2], acc);
                }
            }
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    along(I0{}, I1{}, I2{}, s.cx);
    along(I1{}, I0{}, I2{}, s.cy);
    if (DIM == 3) {
        along(I2{}, I0{}, I1{}, s.cz);
    } else if (s.cz != 0.0f) {
        for (int j = 0; j < 3; ++j)
            for (int i = 0; i < 3; ++i) {
                const float wt = cross_factor(s.S0[0][i], s.D[0][i], s.S0[1][j], s.D[1][j]);
                if (ALL || wt != 0.0f) add(2, i, j, 0, s.cz * wt);
            }
    }
}

template <int DIM>
__global__ __launch_bounds__(kDepThreads) __attribute__((amdgpu_waves_per_eu(6))) void current_kernel(sr_particles_f32 P, const float *xo0,
                                                      const float *xo1, const float *xo2,
                                                      PicGrid G, float qv, float inv_dt,
                                                      float *__restrict__ jx, float *__restrict__ jy,
                                                      float *__restrict__ jz,
                                                      uint32_t *__restrict__ status, int max_slabs) {
    __shared__ int box[3 * kDepCells];
    __shared__ uint32_t row[kDepRows];
    __shared__ uint16_t list[kDepThreads];
    __shared__ int listed;
    __shared__ float bsum[kDepThreads / 64];
    __shared__ DepShared sh;
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool active = p < P.n;
    const uint32_t u = active ? (uint32_t)p : 0u;
    const float *const xo[3] = {xo0, xo1, xo2};
    bool bad;
    const Move m = make_move<DIM>(P, xo, G, qv, inv_dt, u, active, bad);
    if (bad) atomicOr(status, SR_W_CFL);
    float *const J[3] = {jx, jy, jz};

    // the block's first particle is always active: the grid has
    // ceil(n / kDepThreads) blocks
    int U[3];
    DepBox bx;
    if (!deposit_box<DIM, true>(sh, m.I, m.live, m.bound, G, 1, 2, kDepCells, max_slabs, U, bx))
        return;                     // no live particle (the condition is block-wide)
    const float bnd = bx.bnd;
    if (!(bnd > 0.0f)) return;      // block-wide: every contribution is zero
    // bnd < 2^e: contributions in units of 2^(e - kDepFracBits).  A
    // non-finite bound, or one so small that 2^(kDepFracBits - e) would not
    // be a finite float, sends the whole block to the float path; in slabs so does one
    // whose sums or scale might not be.
    int e = 0;
    (void)frexpf(bnd, &e);
    const bool fixed = bx.slabs == 1 ? bnd <= 3.0e38f && e >= -100 : e <= 115 && e >= -80;
    if (!fixed) bx.slabs = 1;
    float to_fix = fixed ? ldexpf(1.0f, kDepFracBits - e) : 0.0f;
    float from_fix = fixed ? ldexpf(1.0f, e - kDepFracBits) : 0.0f;
    float least = 0.0f;
    const bool in_cell = m.live && fixed && stays<DIM>(m);
    for (int t = 0; t < bx.slabs; ++t) {
        DepBox w;
        const bool mine = deposit_slab<DIM>(bx, t, 1, 2, U, w);
        const int cells = w.ext[0] * w.ext[1] * w.ext[2];
        const int e0 = w.ext[0], e01 = w.ext[0] * w.ext[1];
        if (t) __syncthreads();        // the box is flushed, the list is read
        if (threadIdx.x == 0) listed = 0;
        if (bx.slabs > 1) {
            const float b = wave_sum_f(m.live && mine ? m.bound : 0.0f);
            if ((threadIdx.x & 63) == 0) bsum[threadIdx.x >> 6] = b;
        }
        if (fixed) {
            for (int q = threadIdx.x; q < 3 * cells; q += kDepThreads) box[q] = 0;
            box_rows<DIM>(row, w, G);
        }
        __syncthreads();
        if (bx.slabs > 1) {
            float sum_b = 0.0f;
#pragma unroll
            for (int q = 0; q < kDepThreads / 64; ++q) sum_b += bsum[q];
            (void)frexpf(fmaxf(sum_b, 0x1p-82f), &e);
            to_fix = ldexpf(1.0f, kDepSumBits - e);
            from_fix = ldexpf(1.0f, e - kDepSumBits);
            least = sum_b * kDepLight;
        }
        bool now = in_cell && mine && m.bound >= least;
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
            // (the general stencil's nodes, so that a window holds the same particles)
            const int b = U[a] - w.org[a];
            now = now && b >= 0 && b + 2 <= w.ext[a] - 1;
        }
        if (now) {
            const int l0 = (U[0] - w.org[0]) + e0 * (U[1] - w.org[1]) +
                           (DIM == 3 ? e01 * (U[2] - w.org[2]) : 0);
            esirkepov_stay<DIM>(m, [&](int comp, int ci, int cj, int ck, float v) {
                atomicAdd(&box[comp * cells + l0 + ci + (cj ? e0 : 0) + (ck ? e01 : 0)],
                          __float2int_rn(v * to_fix));
            });
        }
        // the slab's others, listed
        {
            const bool later = m.live && mine && !now;
            const uint64_t mask = __ballot(later);
            int base = 0;
            if (mask && (threadIdx.x & 63) == 0) base = atomicAdd(&listed, (int)__popcll(mask));
            base = __builtin_amdgcn_readfirstlane(base);
            if (later) list[base + lane_prefix(mask)] = (uint16_t)threadIdx.x;
        }
        __syncthreads();
        const int n_list = listed;
        for (int q = threadIdx.x; q < n_list; q += kDepThreads) {
            bool unused;
            const uint32_t v = (uint32_t)((int64_t)blockIdx.x * kDepThreads + list[q]);
            const Move y = make_move<DIM>(P, xo, G, qv, inv_dt, v, true, unused);
            const Stencil s = make_stencil<DIM>(y);
            bool in_win = fixed && y.bound >= least;
            int B[3] = {0, 0, 0};
#pragma unroll
            for (int a = 0; a < DIM; ++a) {
                B[a] = unwrap_cell(y.I[a], sh.ref[a], G.n[a]) - 1 + s.o[a] - w.org[a];
                in_win = in_win && B[a] >= 0 && B[a] + 2 <= w.ext[a] - 1;
            }
            if (in_win)
                esirkepov<DIM, true>(s, [&](int c, int ci, int cj, int ck, float x) {
                    const int l = (B[0] + ci) + e0 * (B[1] + cj) + e01 * (B[2] + ck);
                    atomicAdd(&box[c * cells + l], __float2int_rn(x * to_fix));
                });
            else
                esirkepov<DIM, false>(s, [&](int c, int ci, int cj, int ck, float x) {
                    const int i = node(y.I[0], s.o[0] + ci, G.n[0]);
                    const int j = node(y.I[1], s.o[1] + cj, G.n[1]);
                    const int k = DIM == 3 ? node(y.I[2], s.o[2] + ck, G.n[2]) : 0;
                    unsafeAtomicAdd(&J[c][cell(i, j, k, G)], x);
                });
        }
        __syncthreads();
        if (!fixed) return;             // block-wide (one slab: its list held every particle)
        const float inv_e0 = 1.0f / (float)e0;
        for (int q = threadIdx.x; q < cells; q += kDepThreads) {
            int sum[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) sum[c] = box[c * cells + q];
            if ((sum[0] | sum[1] | sum[2]) == 0) continue;
            const uint32_t at = box_node(q, row, w, inv_e0, G);
#pragma unroll
            for (int c = 0; c < 3; ++c)
                if (sum[c] != 0) unsafeAtomicAdd(&J[c][at], (float)sum[c] * from_fix);
        }
    }
}

// Photons move at c along their direction: pos += dt dir, wrapped into the box
// (one lane per chunk segment, as the photon histograms).
__global__ __launch_bounds__(256) void photon_advance_kernel(sr_photon_buf ph, const int64_t *start,
                                                             int64_t n_chunks, int64_t n, PicGrid G,
                                                             int dim, float dt) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n_chunks) return;
    const int64_t s0 = start ? start[c] : c * (int64_t)kChunk;
    const int64_t e0 = start ? start[c + 1] : min(s0 + (int64_t)kChunk, n);
    const int64_t cap = (e0 - s0) * ph.per_particle;
    const int64_t cnt = min((int64_t)ph.seg_count[c], cap);
    const int64_t base = s0 * ph.per_particle;
    for (int64_t q = 0; q < cnt; ++q) {
        const uint32_t o = (uint32_t)(base + q);
        for (int a = 0; a < 3; ++a) {
            if (!ph.pos[a]) continue;
            float v = fmaf(dt, ld(ph.dir[a], o), ld(ph.pos[a], o));
            if (a < dim) {
                const float L = G.L[a];
                v -= L * floorf(v / L);
                if (v >= L || v < 0.0f) v = 0.0f;   // rounding guard (and a corrupt value)
            }
            st(ph.pos[a], o, v);
        }
    }
}

}  // namespace
}  // namespace sr

using namespace sr;

extern "C" int sr_field_step(float *e[3], float *b[3], const float *j[3], const sr_grid *grid,
                             double dt, void *stream) {
    PicGrid G;
    const int rc = pic_grid(grid, G);
    if (rc != SR_OK) return rc;
    if (!e || !b) return SR_E_INVAL;
    for (int q = 0; q < 3; ++q)
        if (!e[q] || !b[q]) return SR_E_INVAL;
    const bool has_j = j && j[0];
    if (has_j && (!j[1] || !j[2])) return SR_E_INVAL;
    // Courant condition of the Yee scheme: dt^2 (sum 1/dx_a^2) < 1
    double s = 0.0;
    for (int a = 0; a < grid->dim; ++a) s += 1.0 / (grid->dx[a] * grid->dx[a]);
    if (!(dt > 0.0) || !(dt * dt * s < 1.0)) return SR_E_INVAL;
    const uint32_t cells = (uint32_t)(grid->n[0] * grid->n[1] * grid->n[2]);
    const unsigned nb = (cells + 255) / 256;
    hipStream_t st = (hipStream_t)stream;
    const float h[3] = {(float)(0.5 * dt / grid->dx[0]), (float)(0.5 * dt / grid->dx[1]),
                        grid->dim == 3 ? (float)(0.5 * dt / grid->dx[2]) : 0.0f};
    const float t[3] = {2.0f * h[0], 2.0f * h[1], 2.0f * h[2]};
    for (int half = 0; half < 3; ++half) {
        if (half == 1) {
            if (grid->dim == 3) {
                if (has_j) curl_b_kernel<3, true><<<nb, 256, 0, st>>>(e[0], e[1], e[2], b[0], b[1], b[2], j[0], j[1], j[2], G, (float)dt, t[0], t[1], t[2], cells);
                else curl_b_kernel<3, false><<<nb, 256, 0, st>>>(e[0], e[1], e[2], b[0], b[1], b[2], nullptr, nullptr, nullptr, G, (float)dt, t[0], t[1], t[2], cells);
            } else {
                if (has_j) curl_b_kernel<2, true><<<nb, 256, 0, st>>>(e[0], e[1], e[2], b[0], b[1], b[2], j[0], j[1], j[2], G, (float)dt, t[0], t[1], t[2], cells);
                else curl_b_kernel<2, false><<<nb, 256, 0, st>>>(e[0], e[1], e[2], b[0], b[1], b[2], nullptr, nullptr, nullptr, G, (float)dt, t[0], t[1], t[2], cells);
            }
        } else {
            if (grid->dim == 3)
                curl_e_kernel<3><<<nb, 256, 0, st>>>(e[0], e[1], e[2], b[0], b[1], b[2], G, h[0], h[1], h[2], cells);
            else
                curl_e_kernel<2><<<nb, 256, 0, st>>>(e[0], e[1], e[2], b[0], b[1], b[2], G, h[0], h[1], h[2], cells);
        }
    }
    SR_HIP_CHECK(hipGetLastError());
    return SR_OK;
}

extern "C" int sr_deposit_rho(const sr_particles_f32 *parts, const sr_grid *grid, double charge,
                              float *rho, void *stream) {
    PicGrid G;
    const int rc = pic_grid(grid, G);
    if (rc != SR_OK) return rc;
    if (!parts || !rho || parts->n < 0) return SR_E_INVAL;
    // element offsets are formed as 32-bit byte offsets (below 2^31 bytes)
    if (parts->n >= ((int64_t)1 << 29)) return SR_E_UNSUPPORTED;
    if (parts->n == 0) return SR_OK;
    if (!parts->x[0] || !parts->x[1] || (grid->dim == 3 && !parts->x[2]) || !parts->w)
        return SR_E_INVAL;
    const unsigned nb = (unsigned)((parts->n + kRhoThreads - 1) / kRhoThreads);
    hipStream_t st = (hipStream_t)stream;
    const int slabs = rho_slabs(parts->n, grid->dim, (double)G.n[0] * G.n[1] * G.n[2]);
    const float qv = (float)charge;
    if (grid->dim == 3) {
        if (slabs) rho_kernel<3><<<nb, kRhoThreads, 0, st>>>(*parts, G, qv, rho, slabs);
        else rho_direct_kernel<3><<<nb, kRhoThreads, 0, st>>>(*parts, G, qv, rho);
    } else {
        if (slabs) rho_kernel<2><<<nb, kRhoThreads, 0, st>>>(*parts, G, qv, rho, slabs);
        else rho_direct_kernel<2><<<nb, kRhoThreads, 0, st>>>(*parts, G, qv, rho);
    }
    SR_HIP_CHECK(hipGetLastError());
    return SR_OK;
}

extern "C" int sr_deposit_current(const sr_particles_f32 *parts, const float *x_old[3],
                                  const sr_grid *grid, double dt, double charge, float *j[3],
                                  uint32_t *status, void *stream) {
    PicGrid G;
    const int rc = pic_grid(grid, G);
    if (rc != SR_OK) return rc;
    if (!parts || !x_old || !j || !status || !(dt > 0.0) || parts->n < 0) return SR_E_INVAL;
    // element offsets are formed as 32-bit byte offsets (below 2^31 bytes)
    if (parts->n >= ((int64_t)1 << 29)) return SR_E_UNSUPPORTED;
    for (int q = 0; q < 3; ++q)
        if (!j[q]) return SR_E_INVAL;
    if (parts->n == 0) return SR_OK;
    const int dim = grid->dim;
    for (int a = 0; a < dim; ++a)
        if (!parts->x[a] || !x_old[a]) return SR_E_INVAL;
    if (!parts->w || (dim == 2 && (!parts->p[0] || !parts->p[1] || !parts->p[2])))
        return SR_E_INVAL;
    const unsigned nb = (unsigned)((parts->n + kDepThreads - 1) / kDepThreads);
    const int slabs = current_slabs(parts->n, dim);
    hipStream_t st = (hipStream_t)stream;
    if (dim == 3)
        current_kernel<3><<<nb, kDepThreads, 0, st>>>(*parts, x_old[0], x_old[1], x_old[2], G, (float)charge,
                                              (float)(1.0 / dt), j[0], j[1], j[2], status, slabs);
    else
        current_kernel<2><<<nb, kDepThreads, 0, st>>>(*parts, x_old[0], x_old[1], nullptr, G, (float)charge,
                                              (float)(1.0 / dt), j[0], j[1], j[2], status, slabs);
    SR_HIP_CHECK(hipGetLastError());
    return SR_OK;
}

extern "C" int sr_photon_advance(const sr_photon_buf *ph, const sr_chunking *chunks, int64_t n,
                                 const sr_grid *grid, double dt, void *stream) {
    PicGrid G;
    const int rc = pic_grid(grid, G);
    if (rc != SR_OK) return rc;
    if (!ph || !chunks || n < 0 || !ph->seg_count || !(dt >= 0.0)) return SR_E_INVAL;
    const int64_t n_chunks = chunks->start ? chunks->n_chunks : (n + kChunk - 1) / kChunk;
    if (n_chunks == 0 || ph->per_particle == 0) return SR_OK;
    if (!ph->dir[0] || !ph->dir[1] || !ph->dir[2]) return SR_E_INVAL;
    // photon slots are addressed with 32-bit byte offsets (below 2^32 bytes)
    if (n * ph->per_particle >= ((int64_t)1 << 30)) return SR_E_UNSUPPORTED;
    const unsigned nb = (unsigned)((n_chunks + 255) / 256);
    photon_advance_kernel<<<nb, 256, 0, (hipStream_t)stream>>>(*ph, chunks->start, n_chunks, n, G,
                                                               grid->dim, (float)dt);
    SR_HIP_CHECK(hipGetLastError());
    return SR_OK;
}
