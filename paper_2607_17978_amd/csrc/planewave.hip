// Gaussian-on-grid ("plane-wave") Coulomb operator: the matrix-vector
// product of the paper's eq. matvec evaluated without an Ewald split
// ("Electrostatics Solvers": the charge density is put on a uniform grid,
// Fourier transformed, multiplied by 4 pi / G^2 and transformed back, and the
// potential is integrated over each atom's Gaussian density).
//
//   theta_i(g) = dV rho_i(r_g - r_i)
//              = dV / ((2 pi)^{3/2} sigma_i^3) exp(-|r_g - r_i|^2 / (2 sigma_i^2)),
//   Q(g)       = sum_j src_j theta_j(g)                  (all periodic images)
//   phi        = unnormalised inverse DFT of (4 pi / (V k^2)) DFT(Q), k != 0
//   (A src)_i  = sum_g theta_i(g) phi(g)
//   F_i        = -q_i sum_g theta_i(g) phi(g) (r_g - r_i) / sigma_i^2
//
// theta_i is cut at |r_g - r_i| <= c sigma_i (c = 6 by default: the
// discarded tail changes the operator by ~1e-8 relative at the configs'
// grid spacing).  With the k = 0 term omitted this is the plane-wave
// definition of the periodic Gaussian-charge energy, self interaction and
// neutralising background included, so there is no real-space pair term, no
// self term and no background correction.
//
// Passes per product:
//   1. spread: one wave per 4 x 4 x 4 grid tile, a lane per point, over the
//   tile's list of atoms whose support meets it (built once per geometry), the
//   sum in a register; 2. R2C along axis 3 in LDS tiles; 3. the spline path's
//   axis-2 / axis-1 (+ Green's function with eta = 0 and unit moduli) / inverse
//   passes; 4. integration: the same tiles and lists, each entry's 64 products
//   summed over the wave, and a sum over each atom's tiles.
// Against atoms walking their supports (FP32 global atomics in the spread, a
// gather per atom in the integration): 4,096 atoms on 96^3, spread 87 + 4 (zero
// fill) -> 21 us, integration 47 -> 31 us (a solve 9.2 -> 3.5 ms), and the sums have one
// order.  Where the lists do not fit (PW_ENT_MAX entries) the walks remain: one
// wave per atom, the points of one grid plane of the support ellipsoid's
// bounding box spread over the lanes with an incremental (row, column) counter,
// so that no lane divides per point.  The final product with forces always
// walks.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "internal.h"
#include "mesh_len.h"

namespace {

constexpr int PW_NT = 256;
constexpr double PW_PI = 3.14159265358979323846;
constexpr float PW_LOG2E = 1.4426950408889634f;

__device__ __forceinline__ int pw_wrap(int g, int K) {
    if (g >= 0 && g < K) return g;
    const int m = g % K;
    return m < 0 ? m + K : m;
}

// Cross-section of the ellipsoid d^T G d <= R2 with the grid plane at offset
// d1 along axis 1: centre (x2, x3) and half-extents (e2, e3) of its bounding
// box; false when the plane misses it.  (The 2x2 block of G and the extent
// factors are constants of the cell, precomputed on the host.)
__device__ __forceinline__ bool pw_section(const PwGeom& g, float d1, float R2, float& x2, float& x3, float& e2,
                                           float& e3) {
    const float b2 = g.G[3] * d1, b3 = g.G[4] * d1;
    x2 = -(g.G[2] * b2 - g.G[5] * b3) * g.inv_det23;
    x3 = -(g.G[1] * b3 - g.G[5] * b2) * g.inv_det23;
    const float rho2 = R2 - (g.G[0] * d1 * d1 + b2 * x2 + b3 * x3);
    if (!(rho2 >= 0.f)) return false;
    const float rho = sqrtf(rho2);
    e2 = rho * g.ext2;
    e3 = rho * g.ext3;
    return true;
}

// Per-atom constants: integer cell of the atom on the grid, fractional offset
// inside it, and the Gaussian's parameters.
struct PwAtom {
    int fl[3];
    float du[3];
    float R2;    // (c sigma)^2 in bohr^2
    float lsc;   // log2(e) / (2 sigma^2)
};

__device__ __forceinline__ PwAtom pw_atom(const KParams& k, const PwGeom& g, const double* frac, double s, int i) {
    PwAtom a;
    const int Kd[3] = {k.K1, k.K2, k.K3};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double u = frac[3 * i + c] * (double)Kd[c];
        const double f = floor(u);
        a.fl[c] = (int)f;
        a.du[c] = (float)(u - f);
    }
    a.R2 = g.c2 * (float)(s * s);
    a.lsc = PW_LOG2E / (float)(2.0 * s * s);
    // a position the input check rejected: no support (the solve reports EINVAL)
    if (!(isfinite(a.du[0]) && isfinite(a.du[1]) && isfinite(a.du[2]) && a.R2 > 0.f)) {
        a.fl[0] = a.fl[1] = a.fl[2] = 0;
        a.du[0] = a.du[1] = a.du[2] = 0.f;
        a.R2 = 0.f;
    }
    return a;
}

// Walks the support of one atom plane by plane: body(idx, Q, d1, d2, d3) runs
// for every grid point inside the cut sphere (grid index, squared distance
// d^T G d, offsets in grid steps), the points spread over the lanes.
template <typename Body>
__device__ __forceinline__ void pw_walk(const KParams& k, const PwGeom& g, const PwAtom& a, int lane, Body body) {
    if (!(a.R2 > 0.f)) return;
    const float e1 = sqrtf(a.R2) * g.ext1;
    const int t1lo = (int)ceilf(a.du[0] - e1), t1hi = (int)floorf(a.du[0] + e1);
    for (int t1 = t1lo; t1 <= t1hi; ++t1) {
        const float d1 = (float)t1 - a.du[0];
        float x2, x3, e2, e3;
        if (!pw_section(g, d1, a.R2, x2, x3, e2, e3)) continue;
        const int t2lo = (int)ceilf(x2 - e2 + a.du[1]), t2hi = (int)floorf(x2 + e2 + a.du[1]);
        const int t3lo = (int)ceilf(x3 - e3 + a.du[2]), t3hi = (int)floorf(x3 + e3 + a.du[2]);
        const int n2 = t2hi - t2lo + 1, n3 = t3hi - t3lo + 1;
        if (n2 <= 0 || n3 <= 0) continue;
        const size_t pbase = (size_t)pw_wrap(a.fl[0] + t1, k.K1) * k.K2 * k.K3;
        const float c1 = g.G[0] * d1 * d1, l2 = 2.f * g.G[3] * d1, l3 = 2.f * g.G[4] * d1;
        const int nbox = n2 * n3;
        const int dq = 64 / n3, dr = 64 - dq * n3;
        // lane / n3 through the reciprocal: exact for lane < 64 (the quotient
        // is at least 0.5 / n3 away from an integer)
        int qq = (int)(((float)lane + 0.5f) * (1.0f / (float)n3));
        int rr = lane - qq * n3;
        for (int j = lane; j < nbox; j += 64) {
            const int t2 = t2lo + qq, t3 = t3lo + rr;
            const float d2 = (float)t2 - a.du[1], d3 = (float)t3 - a.du[2];
            const float Q = c1 + d2 * (l2 + g.G[1] * d2 + 2.f * g.G[5] * d3) + d3 * (l3 + g.G[2] * d3);
            if (Q <= a.R2) {
                const size_t idx = pbase + (size_t)pw_wrap(a.fl[1] + t2, k.K2) * k.K3 + pw_wrap(a.fl[2] + t3, k.K3);
                body(idx, Q, d1, d2, d3);
            }
            qq += dq;
            rr += dr;
            if (rr >= n3) {
                rr -= n3;
                ++qq;
            }
        }
    }
}

// ------------------------------------------------------------------ tile lists
constexpr int PW_E = 4;                          // points of a tile per axis (K_a % 4 == 0)
constexpr size_t PW_ENT_MAX = (size_t)1 << 28;   // most list entries (9.7 GB)

// Tiles that an atom's support can meet, over the lanes: f(tile index, offsets of
// the tile's first point from the atom's grid cell, order among the atom's
// tiles).  A tile is taken when its centre lies within the support radius plus
// the tile's largest half diagonal (in the metric G): never too few.
template <typename F>
__device__ __forceinline__ int pw_tiles_of(const KParams& k, const PwGeom& g, const PwAtom& a, float hdiag, int lane,
                                           F f) {
    if (!(a.R2 > 0.f)) return 0;
    const float R = sqrtf(a.R2), rr = (R + hdiag) * (R + hdiag) * 1.0001f;
    const float ext[3] = {sqrtf(a.R2) * g.ext1, sqrtf(a.R2) * g.bext2, sqrtf(a.R2) * g.bext3};
    const int Kt[3] = {k.K1 / PW_E, k.K2 / PW_E, k.K3 / PW_E};
    int lo[3], cnt[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const int p0 = a.fl[c] + (int)floorf(a.du[c] - ext[c]), p1 = a.fl[c] + (int)ceilf(a.du[c] + ext[c]);
        lo[c] = (p0 - (((p0 % PW_E) + PW_E) % PW_E)) / PW_E;   // floor(p0 / 4)
        cnt[c] = (p1 - (((p1 % PW_E) + PW_E) % PW_E)) / PW_E - lo[c] + 1;
    }
    const int total = cnt[0] * cnt[1] * cnt[2];
    int found = 0;
    for (int b = 0; b < total; b += 64) {
        const int t = b + lane;
        const int t3 = t % cnt[2], t2 = (t / cnt[2]) % cnt[1], t1 = t / (cnt[2] * cnt[1]);
        const int T[3] = {lo[0] + t1, lo[1] + t2, lo[2] + t3};
        int o[3];
        float d[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            o[c] = T[c] * PW_E - a.fl[c];
            d[c] = (float)o[c] + 0.5f * (PW_E - 1) - a.du[c];
        }
        const float Q = g.G[0] * d[0] * d[0] + g.G[1] * d[1] * d[1] + g.G[2] * d[2] * d[2] +
                        2.f * (g.G[3] * d[0] * d[1] + g.G[4] * d[0] * d[2] + g.G[5] * d[1] * d[2]);
        const bool in = t < total && Q <= rr;
        const unsigned long long m = __ballot(in);
        if (in) {
            const int tile = (pw_wrap(T[0], Kt[0]) * Kt[1] + pw_wrap(T[1], Kt[1])) * Kt[2] + pw_wrap(T[2], Kt[2]);
            f(tile, o, found + __popcll(m & ((1ull << lane) - 1)));
        }
        found += __popcll(m);
    }
    return found;
}

// One wave per atom: its record, its tile count, the tiles' entry counts.
__global__ __launch_bounds__(PW_NT) void k_pw_count(KParams k, PwGeom g, const double* __restrict__ frac,
                                                  const double* __restrict__ sig, float4* __restrict__ rec,
                                                  double* __restrict__ amp, int* __restrict__ acount,
                                                  int* __restrict__ tcount) {
    const int lane = threadIdx.x & 63;
    const int i = (blockIdx.x * PW_NT + threadIdx.x) >> 6;
    if (i >= k.n) return;
    const double s = sig[i];
    const PwAtom a = pw_atom(k, g, frac, s, i);
    const int c = pw_tiles_of(k, g, a, g.hdiag, lane, [&](int tile, const int*, int) { atomicAdd(tcount + tile, 1); });
    if (lane == 0) {
        rec[i] = make_float4(a.du[0], a.du[1], a.du[2], a.lsc);
        amp[i] = (double)g.wpref / (s * s * s);
        acount[i] = c;
    }
}

__global__ __launch_bounds__(PW_NT) void k_pw_fill(KParams k, PwGeom g, const double* __restrict__ frac,
                                                 const double* __restrict__ sig, const int* __restrict__ astart,
                                                 const int* __restrict__ tstart, int* __restrict__ cursor,
                                                 int4* __restrict__ ent) {
    const int lane = threadIdx.x & 63;
    const int i = (blockIdx.x * PW_NT + threadIdx.x) >> 6;
    if (i >= k.n) return;
    const PwAtom a = pw_atom(k, g, frac, sig[i], i);
    const int slot0 = astart[i];
    pw_tiles_of(k, g, a, g.hdiag, lane, [&](int tile, const int* o, int order) {
        // offsets stay within four grid lengths (the support check of the set-up)
        const int at = tstart[tile] + atomicAdd(cursor + tile, 1);
        ent[at] = make_int4(i, (o[0] & 0xffff) | (o[1] << 16), o[2], slot0 + order);
    });
}

// One wave per tile: its entries in slot order (so by atom), whatever order the
// fill's cursor gave them.  Short lists by rank within the wave, long ones by
// rank over global memory.
__global__ __launch_bounds__(PW_NT) void k_pw_order(int ntiles, const int* __restrict__ tstart,
                                                  const int4* __restrict__ in, int4* __restrict__ out) {
    const int lane = threadIdx.x & 63;
    const int tile = (blockIdx.x * PW_NT + threadIdx.x) >> 6;
    if (tile >= ntiles) return;
    const int e0 = tstart[tile], cnt = tstart[tile + 1] - e0;
    for (int b = 0; b < cnt; b += 64) {
        const bool live = b + lane < cnt;
        const int4 mine = live ? in[e0 + b + lane] : make_int4(0, 0, 0, 0);
        int rank = 0;
        for (int c = 0; c < cnt; c += 64) {
            const int other = c + lane < cnt ? in[e0 + c + lane].w : 0x7fffffff;
            const int m = min(64, cnt - c);
            for (int t = 0; t < m; ++t) rank += __shfl(other, t, 64) < mine.w ? 1 : 0;
        }
        if (live) out[e0 + rank] = mine;
    }
}

// Records of up to 64 entries of a tile, one per lane, in the wave's LDS: offsets
// of the tile from the atom, the atom's fraction and exponent, R^2 and amplitude.
struct PwRec {
    float4 o;   // offsets 1, 2, 3, (c sigma)^2
    float4 d;   // fractions 1, 2, 3, log2(e) / (2 sigma^2)
    float amp;
    int slot;
    float pad[2];
};

__device__ __forceinline__ void pw_stage(const int4* ent, int e, bool live, const float4* rec, const double* amp,
                                         const double* src, float c2, PwRec* out) {
    if (!live) return;
    const int4 t = ent[e];
    PwRec r;
    r.d = rec[t.x];
    // (c sigma)^2 from the exponent: c^2 log2(e) / (2 lsc)
    r.o = make_float4((float)(short)(t.y & 0xffff), (float)(t.y >> 16), (float)t.z, c2 * (0.5f * PW_LOG2E) / r.d.w);
    r.amp = src ? (float)(src[t.x] * amp[t.x]) : 0.f;
    r.slot = t.w;
    *out = r;
}

// theta / amplitude of an entry at the lane's point (0 outside the support).
template <bool ORTHO>
__device__ __forceinline__ float pw_theta(const PwGeom& g, const PwRec& r, float a1, float a2, float a3) {
    const float d1 = (r.o.x + a1) - r.d.x, d2 = (r.o.y + a2) - r.d.y, d3 = (r.o.z + a3) - r.d.z;
    float Q;
    if (ORTHO)
        Q = g.G[0] * d1 * d1 + (g.G[1] * d2 * d2 + g.G[2] * d3 * d3);
    else
        Q = g.G[0] * d1 * d1 + d2 * (2.f * g.G[3] * d1 + g.G[1] * d2 + 2.f * g.G[5] * d3) +
            d3 * (2.f * g.G[4] * d1 + g.G[2] * d3);
    const float e = __builtin_amdgcn_exp2f(-Q * r.d.w);
    return Q <= r.o.w ? e : 0.f;
}

// One wave per tile, a lane per point: Q(g) = sum over the tile's entries.
// VALU-bound: about 20 instructions per entry and wave, 39 entries per tile at
// 0.01 atoms per bohr^3 (30 of them reach a given point).
template <bool ORTHO>
__global__ __launch_bounds__(PW_NT) void k_pw_tile_spread(KParams k, PwGeom g, int ntiles,
                                                        const int* __restrict__ tstart, const int4* __restrict__ ent,
                                                        const float4* __restrict__ rec, const double* __restrict__ amp,
                                                        const double* __restrict__ src, float* __restrict__ grid,
                                                        const int* __restrict__ done) {
    if (done && *done) return;
    __shared__ PwRec recs[PW_NT / 64][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int tile = xcd_remap(blockIdx.x, gridDim.x) * (PW_NT / 64) + w;
    if (tile >= ntiles) return;   // whole waves; no block barriers below
    const int e0 = tstart[tile], e1 = tstart[tile + 1];
    const float a1 = (float)(lane >> 4), a2 = (float)((lane >> 2) & 3), a3 = (float)(lane & 3);
    float q = 0.f;
    for (int e = e0; e < e1; e += 64) {
        const int m = min(64, e1 - e);
        wave_exchange();
        pw_stage(ent, e + lane, lane < m, rec, amp, src, g.c2, &recs[w][lane]);
        wave_exchange();
#pragma unroll 4
        for (int t = 0; t < m; ++t) {
            const PwRec& r = recs[w][t];
            q += r.amp * pw_theta<ORTHO>(g, r, a1, a2, a3);
        }
    }
    const int Kt2 = k.K2 / PW_E, Kt3 = k.K3 / PW_E;
    const int T3 = tile % Kt3, T2 = (tile / Kt3) % Kt2, T1 = tile / (Kt3 * Kt2);
    grid[((size_t)(T1 * PW_E + (lane >> 4)) * k.K2 + T2 * PW_E + ((lane >> 2) & 3)) * k.K3 + T3 * PW_E + (lane & 3)] = q;
}

// The integration's part of a tile: part[slot] = sum over the tile's points of
// theta phi / amplitude.  An entry's products are added within each row of 16
// lanes; lane t of every row keeps entry t of 16, and two exchanges add the four
// rows of all 16 (exchanging the entries' products by halving, 32 at a time, took
// 140 registers and 190 us at 4,096 atoms).
template <bool ORTHO>
__global__ __launch_bounds__(PW_NT) void k_pw_tile_interp(KParams k, PwGeom g, int ntiles,
                                                        const int* __restrict__ tstart, const int4* __restrict__ ent,
                                                        const float4* __restrict__ rec, const float* __restrict__ grid,
                                                        float* __restrict__ part, const int* __restrict__ done) {
    if (done && *done) return;
    __shared__ PwRec recs[PW_NT / 64][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int tile = xcd_remap(blockIdx.x, gridDim.x) * (PW_NT / 64) + w;
    if (tile >= ntiles) return;
    const int e0 = tstart[tile], e1 = tstart[tile + 1];
    const float a1 = (float)(lane >> 4), a2 = (float)((lane >> 2) & 3), a3 = (float)(lane & 3);
    const int Kt2 = k.K2 / PW_E, Kt3 = k.K3 / PW_E;
    const int T3 = tile % Kt3, T2 = (tile / Kt3) % Kt2, T1 = tile / (Kt3 * Kt2);
    const float phi =
        grid[((size_t)(T1 * PW_E + (lane >> 4)) * k.K2 + T2 * PW_E + ((lane >> 2) & 3)) * k.K3 + T3 * PW_E + (lane & 3)];
    for (int e = e0; e < e1; e += 64) {
        const int m = min(64, e1 - e);
        wave_exchange();
        pw_stage(ent, e + lane, lane < m, rec, nullptr, nullptr, g.c2, &recs[w][lane]);
        wave_exchange();
        for (int b = 0; b < m; b += 16) {
            float keep = 0.f;
#pragma unroll 4
            for (int t = 0; t < 16; ++t) {
                if (b + t >= m) break;   // uniform
                const float x = row16_sum(phi * pw_theta<ORTHO>(g, recs[w][b + t], a1, a2, a3));
                keep = (lane & 15) == t ? x : keep;
            }
            keep += __shfl_xor(keep, 16, 64);
            keep += __shfl_xor(keep, 32, 64);
            if (lane < 16 && b + lane < m) part[recs[w][b + lane].slot] = keep;
        }
    }
}

// y_i = amplitude sum over the atom's tiles, 16 lanes per atom.
__global__ __launch_bounds__(PW_NT) void k_pw_tile_sum(int n, const int* __restrict__ astart,
                                                     const float* __restrict__ part, const double* __restrict__ amp,
                                                     double* __restrict__ y, const int* __restrict__ done) {
    if (done && *done) return;
    const int l = threadIdx.x & 15, i = (blockIdx.x * PW_NT + threadIdx.x) >> 4;
    double v = 0.0;
    if (i < n) {
        const int e1 = astart[i + 1];
#pragma unroll 4
        for (int e = astart[i] + l; e < e1; e += 16) v += (double)part[e];
    }
    v = row16_sum(v);
    if (i < n && l == 0) y[i] = amp[i] * v;
}

__global__ __launch_bounds__(PW_NT) void k_pw_clear(int* __restrict__ x, size_t m) {
    const size_t t = (size_t)blockIdx.x * PW_NT + threadIdx.x;
    if (t < m) x[t] = 0;
}

__global__ __launch_bounds__(PW_NT) void k_pw_zero(float4* __restrict__ grid, size_t n4, const int* __restrict__ done) {
    if (done && *done) return;
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n4) grid[t] = make_float4(0.f, 0.f, 0.f, 0.f);
}

// Q(g) += src_i theta_i(g), one wave per atom (sorted order).
__global__ __launch_bounds__(PW_NT) void k_pw_spread(KParams k, PwGeom g, const double* __restrict__ src,
                                                   const double* __restrict__ frac, const double* __restrict__ sig,
                                                   float* __restrict__ grid, const int* __restrict__ done) {
    if (done && *done) return;
    const int lane = threadIdx.x & 63;
    const int nwaves = gridDim.x * (PW_NT / 64);
    const int w0 = (xcd_remap(blockIdx.x, gridDim.x) * PW_NT + threadIdx.x) >> 6;
    for (int i = w0; i < k.n; i += nwaves) {
        const double q = src[i];
        if (q == 0.0) continue;
        const double s = sig[i];
        const PwAtom a = pw_atom(k, g, frac, s, i);
        const float amp = (float)(q * (double)g.wpref / (s * s * s));
        pw_walk(k, g, a, lane, [&](size_t idx, float Q, float, float, float) {
            unsafeAtomicAdd(grid + idx, amp * __builtin_amdgcn_exp2f(-Q * a.lsc));
        });
    }
}

// Axis-3 FFT of the tile in LDS (two real rows packed per complex column,
// acc[g3][row] viewed as buf[g3][row pair]) and the half spectra written
// transposed, C[m3][g1][g2] (m2 contiguous).
__device__ __forceinline__ void pw_tile_r2c(const KParams& k, const FftAxis& ax3, float2* buf, const float2* tw,
                                            int g1, int g20, int W, float2* __restrict__ C, int tid) {
    const int K1 = k.K1, K2 = k.K2, K3 = k.K3, TW = k.TW, ncol = TW >> 1;
    int twl = 0;
    while ((1 << twl) < TW) ++twl;
    fft_lds(buf, ax3, twl - 1, tw, false, tid, PW_NT);
    __syncthreads();
    const int K3h = K3 / 2 + 1;
    for (int t = tid; t < K3h * TW; t += PW_NT) {
        const int r = t & (TW - 1);
        const int m = t >> twl;
        if (r >= W) continue;
        const int pr = r >> 1;
        const float2 Z = buf[m * ncol + pr];
        float2 Zc = buf[(m == 0 ? 0 : K3 - m) * ncol + pr];
        Zc.y = -Zc.y;
        float2 X;
        if ((r & 1) == 0) {
            X = make_float2(0.5f * (Z.x + Zc.x), 0.5f * (Z.y + Zc.y));
        } else {
            const float2 d = csub(Z, Zc);
            X = make_float2(0.5f * d.y, -0.5f * d.x);
        }
        C[((size_t)m * K1 + g1) * K2 + g20 + r] = X;
    }
}

// Real-to-complex transform along axis 3 of the real grid, block = (g1, tile
// of TW rows g2: the axis-1 / complex-to-real tile, a power of two), two
// real rows packed into one complex column; the half
// spectra are written transposed (C[m3][g1][g2]) as by the spline spread.
__global__ __launch_bounds__(PW_NT) void k_pw_r2c(KParams k, FftAxis ax3, const float* __restrict__ R,
                                                float2* __restrict__ C, const int* __restrict__ done) {
    if (done && *done) return;
    extern __shared__ float2 sm[];
    const int K2 = k.K2, K3 = k.K3, TW = k.TW;
    float2* tw = sm;
    float2* buf = sm + K3;
    float* acc = reinterpret_cast<float*>(buf);
    const int tid = threadIdx.x;
    const int blk = xcd_remap(blockIdx.x, gridDim.x);
    const int g1 = blk / k.ntile;
    // the axis-1 / complex-to-real tiles: uniform, or as equal as possible
    const int t2 = blk - g1 * k.ntile, np = K2 >> 1;
    const int g20 = k.rag ? 2 * (t2 * np / k.ntile) : t2 * TW;
    const int W = k.rag ? 2 * ((t2 + 1) * np / k.ntile) - g20 : TW;
    for (int t = tid; t < K3; t += PW_NT) tw[t] = ax3.tw[t];
    // row index fastest: consecutive lanes write consecutive LDS words (the
    // transposed [g3][row] layout the FFT needs); each lane loads 4 values
    // of its row (K3 % 4 == 0)
    for (int e = tid; e < TW * (K3 >> 2); e += PW_NT) {
        const int r = e & (TW - 1), c4 = e / TW;
        const float4 x = r < W ? *reinterpret_cast<const float4*>(R + ((size_t)g1 * K2 + g20 + r) * K3 + 4 * c4)
                               : make_float4(0.f, 0.f, 0.f, 0.f);
        acc[(4 * c4) * TW + r] = x.x;
        acc[(4 * c4 + 1) * TW + r] = x.y;
        acc[(4 * c4 + 2) * TW + r] = x.z;
        acc[(4 * c4 + 3) * TW + r] = x.w;
    }
    __syncthreads();
    pw_tile_r2c(k, ax3, buf, tw, g1, g20, W, C, tid);
}

// y_i = sum_g theta_i(g) phi(g); with FIN the forces of that product for the
// charges src (both sorted order), one wave per atom.
template <bool FIN>
__global__ __launch_bounds__(PW_NT) void k_pw_interp(KParams k, PwGeom g, const double* __restrict__ src,
                                                   const double* __restrict__ frac, const double* __restrict__ sig,
                                                   const float* __restrict__ grid, double* __restrict__ y,
                                                   double* __restrict__ f, const int* __restrict__ done) {
    if (done && *done) return;
    const int lane = threadIdx.x & 63;
    const int nwaves = gridDim.x * (PW_NT / 64);
    const int w0 = (xcd_remap(blockIdx.x, gridDim.x) * PW_NT + threadIdx.x) >> 6;
    const int rounds = (k.n + nwaves - 1) / nwaves;
    for (int rnd = 0; rnd < rounds; ++rnd) {
        const int i = rnd * nwaves + w0;
        float v[4] = {0.f, 0.f, 0.f, 0.f};
        double s = 1.0;
        if (i < k.n) {
            s = sig[i];
            const PwAtom a = pw_atom(k, g, frac, s, i);
            pw_walk(k, g, a, lane, [&](size_t idx, float Q, float d1, float d2, float d3) {
                const float t = __builtin_amdgcn_exp2f(-Q * a.lsc) * grid[idx];
                v[0] += t;
                if (FIN) {
                    v[1] += t * d1;
                    v[2] += t * d2;
                    v[3] += t * d3;
                }
            });
        }
        double vd[4] = {(double)v[0], 0.0, 0.0, 0.0};
        vd[0] = wave_sum(vd[0]);
        if (FIN) {
#pragma unroll
            for (int c = 1; c < 4; ++c) vd[c] = wave_sum((double)v[c]);
        }
        if (i < k.n && lane == 0) {
            const double amp = (double)g.wpref / (s * s * s);
            y[i] = amp * vd[0];
            if (FIN) {
                // F = -q / sigma^2 sum theta phi (r_g - r_i), r_g - r_i = sum_a d_a H[a] / K_a
                const double pre = -src[i] * amp / (s * s);
                for (int c = 0; c < 3; ++c)
                    f[3 * i + c] = pre * (vd[1] * g.HK[c] + vd[2] * g.HK[3 + c] + vd[3] * g.HK[6 + c]);
            }
        }
    }
}

__global__ void k_pw_add_forces(int n, const double* __restrict__ frec, double* __restrict__ forces) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < 3 * n) forces[t] += frec[t];
}

__global__ __launch_bounds__(PW_NT) void k_pw_sigma_max(int n, const double* __restrict__ sig,
                                                      double* __restrict__ part) {
    __shared__ double sh[PW_NT];
    const int i = blockIdx.x * PW_NT + threadIdx.x;
    sh[threadIdx.x] = i < n ? sig[i] : 0.0;
    __syncthreads();
    for (int w = PW_NT / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) sh[threadIdx.x] = fmax(sh[threadIdx.x], sh[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

template <typename T>
int pw_alloc(T** p, size_t count) {
    if (*p) (void)hipFree(*p);
    *p = nullptr;
    if (hipMalloc((void**)p, sizeof(T) * (count ? count : 1)) != hipSuccess) return QEQ_ENOMEM;
    if (poisonable<T>) debug_poison(*p, sizeof(T) * count);
    return QEQ_OK;
}

int pw_blocks(int n) {
    const int waves = PW_NT / 64;
    const int b = (n + waves - 1) / waves;
    return std::max(1, std::min(b, 2048));
}

bool invert3(const double m[9], double out[9]) {
    const double c00 = m[4] * m[8] - m[5] * m[7], c01 = m[5] * m[6] - m[3] * m[8], c02 = m[3] * m[7] - m[4] * m[6];
    const double det = m[0] * c00 + m[1] * c01 + m[2] * c02;
    if (!(fabs(det) > 0.0)) return false;
    const double id = 1.0 / det;
    out[0] = c00 * id;
    out[1] = (m[2] * m[7] - m[1] * m[8]) * id;
    out[2] = (m[1] * m[5] - m[2] * m[4]) * id;
    out[3] = c01 * id;
    out[4] = (m[0] * m[8] - m[2] * m[6]) * id;
    out[5] = (m[2] * m[3] - m[0] * m[5]) * id;
    out[6] = c02 * id;
    out[7] = (m[1] * m[6] - m[0] * m[7]) * id;
    out[8] = (m[0] * m[4] - m[1] * m[3]) * id;
    return true;
}

}  // namespace

void pw_free(qeq_plan* pl) {
    void* ptrs[] = {pl->pw_ones,   pl->pw_y,      pl->pw_f,      pl->pw_smax, pl->pw_tcount,
                    pl->pw_tstart, pl->pw_acount, pl->pw_astart, pl->pw_rec,  pl->pw_amp,  pl->pw_ent,
                    pl->pw_part};
    for (void* q : ptrs)
        if (q) (void)hipFree(q);
    pl->pw_ent = nullptr;
    pl->pw_part = nullptr;
    pl->pw_tcount = pl->pw_tstart = pl->pw_acount = pl->pw_astart = nullptr;
    pl->pw_rec = nullptr;
    pl->pw_amp = nullptr;
    pl->pw_cap_t = pl->pw_cap_a = pl->pw_cap_e = 0;
    pl->pw_tiles = false;
    pl->pw_ones = nullptr;
    pl->pw_y = pl->pw_f = pl->pw_smax = nullptr;
    pl->pw_cap_n = 0;
    pl->pw_cap_k = 0;
}

// Tile lists of the current geometry (pw_tiles = false, and the walks instead,
// where they have more than PW_ENT_MAX entries or do not fit the free memory;
// the axis-3 pass takes tiles of at most LEN_TW rows).  One host
// synchronisation for their length.
static int pw_build_lists(qeq_plan* pl) {
    const KParams& k = pl->kp;
    if (k.TW > LEN_TW) return QEQ_OK;
    const size_t nt = (size_t)(k.K1 / PW_E) * (k.K2 / PW_E) * (k.K3 / PW_E);
    const GrowBuf rec = {&pl->pw_rec, sizeof(float4), 0, true};
    if (!device_grow(pl->pw_cap_t, nt, {grow_buf(pl->pw_tcount, 1), grow_buf(pl->pw_tstart, 1)}) ||
        !device_grow(pl->pw_cap_a, (size_t)pl->n_max,
                     {grow_buf(pl->pw_acount, 1), grow_buf(pl->pw_astart, 1), rec, grow_buf(pl->pw_amp)}))
        return QEQ_ENOMEM;
    const int nb = (int)(((size_t)k.n * 64 + PW_NT - 1) / PW_NT);
    const unsigned cb = (unsigned)((nt + PW_NT - 1) / PW_NT), ob = (unsigned)((nt * 64 + PW_NT - 1) / PW_NT);
    hipStream_t st = pl->stream;
    // bound on the entries: the bounding box of the widest support, every atom
    // (counts past 2^31 cannot arise below it)
    const double widest = 2.0 * pl->pw_geom.rmax;
    double most = (double)k.n;
    const float be[3] = {pl->pw_geom.ext1, pl->pw_geom.bext2, pl->pw_geom.bext3};
    for (int a = 0; a < 3; ++a) most *= widest * be[a] / PW_E + 3.0;
    if (most > 2.0e9) return QEQ_OK;
    hipLaunchKernelGGL(k_pw_clear, dim3(cb), dim3(PW_NT), 0, st, pl->pw_tcount, nt);
    hipLaunchKernelGGL(k_pw_count, dim3(nb), dim3(PW_NT), 0, st, k, pl->pw_geom, pl->frac, pl->sig,
                       (float4*)pl->pw_rec, pl->pw_amp, pl->pw_acount, pl->pw_tcount);
    QEQ_TRY(launch_scan(pl, pl->pw_tcount, pl->pw_tstart, (int)nt));
    QEQ_TRY(launch_scan(pl, pl->pw_acount, pl->pw_astart, k.n));
    int total = 0;
    QEQ_HIP(hipMemcpyAsync(&total, pl->pw_astart + k.n, sizeof(int), hipMemcpyDeviceToHost, st));
    QEQ_HIP(hipStreamSynchronize(st));
    if (total < 0 || (size_t)total > PW_ENT_MAX) return QEQ_OK;
    // the entries twice: as filled, and in order
    if ((size_t)total > pl->pw_cap_e) {
        const size_t cap = std::min(PW_ENT_MAX, (size_t)total + (size_t)total / 8 + 1024);
        const GrowBuf pairs = {&pl->pw_ent, 2 * sizeof(int4), 0, false};
        if (!device_grow(pl->pw_cap_e, cap, {pairs, grow_buf(pl->pw_part)})) return QEQ_ENOMEM;
    }
    int4* ent = (int4*)pl->pw_ent;
    hipLaunchKernelGGL(k_pw_clear, dim3(cb), dim3(PW_NT), 0, st, pl->pw_tcount, nt);
    hipLaunchKernelGGL(k_pw_fill, dim3(nb), dim3(PW_NT), 0, st, k, pl->pw_geom, pl->frac, pl->sig, pl->pw_astart,
                       pl->pw_tstart, pl->pw_tcount, ent + pl->pw_cap_e);
    hipLaunchKernelGGL(k_pw_order, dim3(ob), dim3(PW_NT), 0, st, (int)nt, pl->pw_tstart, ent + pl->pw_cap_e, ent);
    QEQ_TRY(qeq_check(hipGetLastError()));
    pl->pw_tiles = true;
    return QEQ_OK;
}

// The lists, or the walks where there is no memory for them.
static int pw_lists(qeq_plan* pl) {
    pl->pw_tiles = false;
    const int rc = pw_build_lists(pl);
    if (rc != QEQ_ENOMEM) return rc;
    (void)hipGetLastError();
    return QEQ_OK;
}

// Geometry of the current cell and grid; buffers grown as needed.  One host
// sync (the largest sigma bounds the support, checked against the grid).
int pw_setup(qeq_plan* pl) {
    const KParams& k = pl->kp;
    const size_t kmax = (size_t)std::max({k.K1, k.K2, k.K3});
    if (kmax > pl->pw_cap_k) {
        if (!device_grow(pl->pw_cap_k, kmax, {grow_buf(pl->pw_ones)})) return QEQ_ENOMEM;
        std::vector<float> ones(kmax, 1.0f);
        const int rc = upload(pl, pl->pw_ones, ones.data(), sizeof(float) * kmax);
        if (rc != QEQ_OK) pl->pw_cap_k = 0;
        QEQ_TRY(rc);
    }
    if (pl->n_max > pl->pw_cap_n) {
        const size_t nn = (size_t)pl->n_max;
        QEQ_TRY(pw_alloc(&pl->pw_y, nn));
        QEQ_TRY(pw_alloc(&pl->pw_f, 3 * nn));
        QEQ_TRY(pw_alloc(&pl->pw_smax, (nn + PW_NT - 1) / PW_NT));
        pl->pw_cap_n = pl->n_max;
    }
    const int Kd[3] = {k.K1, k.K2, k.K3};
    double G[9], Gi[9];
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b) {
            double d = 0.0;
            for (int c = 0; c < 3; ++c) d += k.H[a * 3 + c] * k.H[b * 3 + c];
            G[a * 3 + b] = d / ((double)Kd[a] * Kd[b]);
        }
    if (!invert3(G, Gi)) return QEQ_EINVAL;
    PwGeom& g = pl->pw_geom;
    const int o[6][2] = {{0, 0}, {1, 1}, {2, 2}, {0, 1}, {0, 2}, {1, 2}};
    for (int t = 0; t < 6; ++t) g.G[t] = (float)G[o[t][0] * 3 + o[t][1]];
    // extent of d^T G d <= 1 along axis a: sqrt((G^-1)_aa); plane sections
    // use the inverse of the (2, 3) block of G
    const double det23 = G[4] * G[8] - G[5] * G[7];
    g.ext1 = (float)sqrt(Gi[0]);
    g.inv_det23 = (float)(1.0 / det23);
    g.ext2 = (float)sqrt(G[8] / det23);
    g.ext3 = (float)sqrt(G[4] / det23);
    g.bext2 = (float)sqrt(Gi[4]);
    g.bext3 = (float)sqrt(Gi[8]);
    // half diagonal of a tile (first to last point), over its four diagonals
    double hd = 0.0;
    for (int sgn = 0; sgn < 4; ++sgn) {
        const double h[3] = {0.5 * (PW_E - 1), (sgn & 1 ? -0.5 : 0.5) * (PW_E - 1), (sgn & 2 ? -0.5 : 0.5) * (PW_E - 1)};
        double q2 = 0.0;
        for (int a = 0; a < 3; ++a)
            for (int b = 0; b < 3; ++b) q2 += h[a] * h[b] * G[a * 3 + b];
        hd = std::max(hd, q2);
    }
    g.hdiag = (float)(1.0001 * sqrt(hd));
    for (int a = 0; a < 3; ++a)
        for (int c = 0; c < 3; ++c) g.HK[a * 3 + c] = (float)(k.H[a * 3 + c] / Kd[a]);
    g.c2 = (float)(pl->pw_support * pl->pw_support);
    const double dV = k.vol / ((double)k.K1 * k.K2 * k.K3);
    g.wpref = (float)(dV / pow(2.0 * PW_PI, 1.5));
    // the support of the widest atom: at most a few grid lengths per axis
    // (a Gaussian far wider than the cell would visit many images per point)
    const int nb = (k.n + PW_NT - 1) / PW_NT;
    hipLaunchKernelGGL(k_pw_sigma_max, dim3(nb), dim3(PW_NT), 0, pl->stream, k.n, pl->sig, pl->pw_smax);
    QEQ_TRY(qeq_check(hipGetLastError()));
    std::vector<double> smax((size_t)nb);
    QEQ_HIP(hipMemcpyAsync(smax.data(), pl->pw_smax, sizeof(double) * nb, hipMemcpyDeviceToHost, pl->stream));
    QEQ_HIP(hipStreamSynchronize(pl->stream));
    double sm = 0.0;
    for (double v : smax) sm = std::max(sm, v);
    const double R = pl->pw_support * sm;
    g.rmax = (float)R;
    for (int a = 0; a < 3; ++a)
        if (R * sqrt(Gi[a * 4]) > 4.0 * Kd[a]) return QEQ_EPLAN;
    return pw_lists(pl);
}

static int pw_interp_launch(qeq_plan* pl, const double* src, const int* done, bool fin, int nb) {
    const KParams& k = pl->kp;
    if (fin)
        hipLaunchKernelGGL(k_pw_interp<true>, dim3(nb), dim3(PW_NT), 0, pl->stream, k, pl->pw_geom, src, pl->frac,
                           pl->sig, pl->grid_r, pl->pw_y, pl->pw_f, done);
    else
        hipLaunchKernelGGL(k_pw_interp<false>, dim3(nb), dim3(PW_NT), 0, pl->stream, k, pl->pw_geom, src, pl->frac,
                           pl->sig, pl->grid_r, pl->pw_y, pl->pw_f, done);
    return qeq_check(hipGetLastError());
}

// y = A src into pw_y (sorted order); with fin also the forces into pw_f.
int launch_pw_rec(qeq_plan* pl, const double* src, const int* done, bool fin) {
    const KParams& k = pl->kp;
    const size_t sh = sizeof(float2) * ((size_t)k.K3 + (size_t)k.K3 * (k.TW / 2));
    const int nb = pw_blocks(k.n);
    const size_t nreal = (size_t)k.K1 * k.K2 * k.K3;   // a multiple of 4 (K_a % 4 == 0)
    if (pl->pw_tiles) {
        const int nt = (int)(nreal / 64);
        const dim3 tb((unsigned)((nt + PW_NT / 64 - 1) / (PW_NT / 64)));
        const PwGeom& g = pl->pw_geom;
        const bool ortho = g.G[3] == 0.f && g.G[4] == 0.f && g.G[5] == 0.f;
        const int4* ent = (const int4*)pl->pw_ent;
        const float4* rec = (const float4*)pl->pw_rec;
        if (ortho)
            hipLaunchKernelGGL(k_pw_tile_spread<true>, tb, dim3(PW_NT), 0, pl->stream, k, g, nt, pl->pw_tstart, ent, rec,
                               pl->pw_amp, src, pl->grid_r, done);
        else
            hipLaunchKernelGGL(k_pw_tile_spread<false>, tb, dim3(PW_NT), 0, pl->stream, k, g, nt, pl->pw_tstart, ent,
                               rec, pl->pw_amp, src, pl->grid_r, done);
        QEQ_TRY(launch_mesh_r2c(pl, done));
        QEQ_TRY(launch_mesh_from_spectrum(pl, done));
        if (fin) return pw_interp_launch(pl, src, done, fin, nb);
        if (ortho)
            hipLaunchKernelGGL(k_pw_tile_interp<true>, tb, dim3(PW_NT), 0, pl->stream, k, g, nt, pl->pw_tstart, ent, rec,
                               pl->grid_r, pl->pw_part, done);
        else
            hipLaunchKernelGGL(k_pw_tile_interp<false>, tb, dim3(PW_NT), 0, pl->stream, k, g, nt, pl->pw_tstart, ent,
                               rec, pl->grid_r, pl->pw_part, done);
        hipLaunchKernelGGL(k_pw_tile_sum, dim3((unsigned)((k.n * 16 + PW_NT - 1) / PW_NT)), dim3(PW_NT), 0, pl->stream,
                           k.n, pl->pw_astart, pl->pw_part, pl->pw_amp, pl->pw_y, done);
        return qeq_check(hipGetLastError());
    }
    hipLaunchKernelGGL(k_pw_zero, dim3((unsigned)((nreal / 4 + PW_NT - 1) / PW_NT)), dim3(PW_NT), 0, pl->stream,
                       (float4*)pl->grid_r, nreal / 4, done);
    hipLaunchKernelGGL(k_pw_spread, dim3(nb), dim3(PW_NT), 0, pl->stream, k, pl->pw_geom, src, pl->frac, pl->sig,
                       pl->grid_r, done);
    if (sh > 65536)
        QEQ_HIP(hipFuncSetAttribute((const void*)k_pw_r2c, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh));
    hipLaunchKernelGGL(k_pw_r2c, dim3(k.K1 * k.ntile), dim3(PW_NT), sh, pl->stream, k, pl->axes.ax[2],
                       pl->grid_r, pl->grid_c, done);
    QEQ_TRY(qeq_check(hipGetLastError()));
    QEQ_TRY(launch_mesh_from_spectrum(pl, done));
    return pw_interp_launch(pl, src, done, fin, nb);
}

int launch_pw_forces_add(qeq_plan* pl) {
    const int n = pl->kp.n;
    hipLaunchKernelGGL(k_pw_add_forces, dim3(nblocks(3 * n)), dim3(QEQ_BLOCK), 0, pl->stream, n, pl->pw_f,
                       pl->fdst);
    return qeq_check(hipGetLastError());
}
