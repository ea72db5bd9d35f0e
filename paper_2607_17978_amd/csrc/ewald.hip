// Reciprocal part of the periodic operator by direct Ewald summation (SI,
// "Ewald Summation"; the Electrostatics Solvers section's O(N^3/2) solver for
// small cells), in place of the particle mesh:
//
//   (E_rec v)_i = sum_{k in a half space, 0 < |k| <= k_max} w_k
//                 [cos(k.r_i) C_k + sin(k.r_i) S_k],
//   C_k + i S_k = sum_j v_j exp(i k.r_j),   w_k = 2 (4 pi / V) exp(-eta^2 k^2 / 2) / k^2,
//
// with k = 2 pi H^-1 m and k_max where exp(-eta^2 k^2 / 2) = 1e-12.  The
// real-space pairs, the self and background terms and the CG loop are the
// mesh path's (the mesh self-correction is off: the sums are exact).  Forces
// of the final product: F_i = -q_i sum_k w_k k [S_k cos(k.r_i) - C_k sin(k.r_i)].
//
// The phases factorise over the axes, exp(i k.r) = e_a[m_a] e_b[m_b] e_c[m_c]
// with e_x[m] = exp(2 pi i m s_x), so both passes of a product are small
// matrix products on the FP64 matrix instructions.  A "row" is a pair
// (m_a, m_b) of the half space, axis c is the one with the most modes:
//
//   T[row, m_c] = sum_j (v_j e_a e_b)[row, j] e_c[m_c, j]           (k_ew_sf)
//   y_i = Re sum_row (e_a e_b)[row, i] sum_mc F[row, m_c] e_c[m_c, i]  (k_ew_pot)
//
// with F = w (C - i S).  +m_c and -m_c share their real products (e_c at -m is
// the conjugate), so one instruction set serves both.  Sums have one fixed
// order.  Phases, products and sums in FP64.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "internal.h"

namespace {

constexpr int EW_MAX_MODES = 1 << 20;
constexpr int EW_SW = 16;            // waves of a structure-factor block
constexpr int EW_PW = 4;             // waves of a potential block
constexpr int EW_BLOCKS = 1024;      // blocks that the row splits aim at
constexpr int EW_SPLIT_MAX = 16;     // row splits of the potential
constexpr size_t EW_TABLE_MAX = (size_t)256 << 20;   // bytes of the phase table
constexpr double EW_PI = 3.14159265358979323846;

typedef double ew_d4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ ew_d4 ew_mfma(double a, double b, ew_d4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// exp(2 pi i m s): the argument reduced to one turn.
__device__ __forceinline__ double2 ew_phase(int m, double s) {
    double t = (double)m * s;
    t -= rint(t);
    double sn, cs;
    sincospi(2.0 * t, &sn, &cs);
    return make_double2(cs, sn);
}

// Phase of multiple m >= 0 of axis slot x (0: a, 1: b, 2: c) at atom j, from
// the table or, where the table was not laid out, computed in place.
template <bool TAB>
__device__ __forceinline__ double2 ew_axis(const EwGeom& g, const double2* __restrict__ tab,
                                           const double* __restrict__ frac, int n, int x, int m, int j) {
    if (TAB) return tab[(size_t)(g.toff[x] + m) * n + j];
    return ew_phase(m, frac[3 * j + g.ax[x]]);
}

// e_a[a] e_b[b] at atom j; b may be negative (the conjugate).
template <bool TAB>
__device__ __forceinline__ double2 ew_row(const EwGeom& g, const double2* __restrict__ tab,
                                          const double* __restrict__ frac, int n, int4 row, int j) {
    const double2 ea = ew_axis<TAB>(g, tab, frac, n, 0, row.x, j);
    double2 eb = ew_axis<TAB>(g, tab, frac, n, 1, abs(row.y), j);
    if (row.y < 0) eb.y = -eb.y;
    return make_double2(ea.x * eb.x - ea.y * eb.y, ea.x * eb.y + ea.y * eb.x);
}

// Set-up of a cell and geometry: the phase table (blocks below nbt) and the
// weights w+ and w- of every (row, m_c) of the tiles: zero outside the half
// space or the cutoff, and for the padding.
__global__ void k_ew_tables(int n, int nbt, EwGeom g, KParams k, const double* __restrict__ frac,
                            const int4* __restrict__ rows, const int2* __restrict__ units,
                            double2* __restrict__ tab, double2* __restrict__ w) {
    if ((int)blockIdx.x < nbt) {
        const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
        if (t >= (size_t)g.ntab * n) return;
        const int m = (int)(t / n), j = (int)(t - (size_t)m * n);
        const int x = m >= g.toff[2] ? 2 : m >= g.toff[1] ? 1 : 0;
        tab[t] = ew_phase(m - g.toff[x], frac[3 * j + g.ax[x]]);
        return;
    }
    const int u = blockIdx.x - nbt, r = threadIdx.x >> 4, cc = threadIdx.x & 15;
    const int2 un = units[u];
    const int4 row = rows[un.x * 16 + r];
    const int c = un.y * 16 + cc;
    double wv[2] = {0.0, 0.0};
    for (int sg = 0; sg < 2; ++sg) {
        if (row.z < 0 || c > row.z) continue;                            // padding
        if (sg == 1 && (c == 0 || (row.x == 0 && row.y == 0))) continue; // counted with w+
        if (c == 0 && row.x == 0 && row.y == 0) continue;                // k = 0
        int m[3];
        m[g.ax[0]] = row.x;
        m[g.ax[1]] = row.y;
        m[g.ax[2]] = sg ? -c : c;
        double k2 = 0.0;
        for (int q = 0; q < 3; ++q) {
            const double kv =
                2.0 * EW_PI * (k.Hinv[q * 3] * m[0] + k.Hinv[q * 3 + 1] * m[1] + k.Hinv[q * 3 + 2] * m[2]);
            k2 += kv * kv;
        }
        if (k2 <= g.kmax2) wv[sg] = 2.0 * 4.0 * EW_PI / k.vol * exp(-0.5 * k.eta * k.eta * k2) / k2;
    }
    w[(size_t)u * 256 + threadIdx.x] = make_double2(wv[0], wv[1]);
}

// Structure factors of one unit (16 rows x 16 m_c): the waves share the
// atoms, four a matrix instruction, and add up through LDS; the weighted
// combinations F+ + F- and F+ - F- go out as operands of k_ew_pot.
// 64 units at 512 atoms: bound by the latency of one unit (three dependent
// loads, 32 matrix instructions a wave, the LDS sum), 12 us where a thread per
// mode with a sine and cosine per (mode, atom) and product took 11; with the
// atoms split over blocks as well this pass lost 3 us and the next gained 4.
// 4,096 atoms (445 units): 165 us, 22 TFLOP/s FP64, bound by the scattered
// 16-byte phase loads.
template <bool TAB>
__global__ __launch_bounds__(64 * EW_SW) void k_ew_sf(int n, EwGeom g, const int4* __restrict__ rows,
                                                      const int2* __restrict__ units, const int2* __restrict__ tiles,
                                                      const double2* __restrict__ tab,
                                                      const double* __restrict__ frac,
                                                      const double2* __restrict__ w, const double* __restrict__ src,
                                                      double* __restrict__ F, const int* __restrict__ done) {
    if (done && *done) return;
    __shared__ double red[EW_SW / 2][1024];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int r = lane & 15, kq = lane >> 4;
    const int2 un = units[blockIdx.x];
    const int4 row = rows[un.x * 16 + r];
    const int c = min(un.y * 16 + r, g.lim[2]);
    const int nk = (n + 3) >> 2, per = (nk + EW_SW - 1) / EW_SW;
    const int k0 = wv * per, k1 = min(nk, k0 + per);
    ew_d4 rc = {0, 0, 0, 0}, ic = rc, rs = rc, is = rc;
#pragma unroll 8
    for (int ks = k0; ks < k1; ++ks) {
        const int j = ks * 4 + kq, jc = min(j, n - 1);
        const double v = j < n ? src[jc] : 0.0;
        const double2 e = ew_row<TAB>(g, tab, frac, n, row, jc);
        const double2 ec = ew_axis<TAB>(g, tab, frac, n, 2, c, jc);
        const double ar = v * e.x, ai = v * e.y;
        rc = ew_mfma(ar, ec.x, rc);
        ic = ew_mfma(ai, ec.x, ic);
        rs = ew_mfma(ar, ec.y, rs);
        is = ew_mfma(ai, ec.y, is);
    }
    // result layout: lane l holds rows l/16 + 4 j of column l%16
    if (wv >= EW_SW / 2) {
        double* d = red[wv - EW_SW / 2];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            d[lane + 64 * j] = rc[j];
            d[256 + lane + 64 * j] = ic[j];
            d[512 + lane + 64 * j] = rs[j];
            d[768 + lane + 64 * j] = is[j];
        }
    }
    __syncthreads();
    if (wv < EW_SW / 2) {
        double* d = red[wv];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            d[lane + 64 * j] += rc[j];
            d[256 + lane + 64 * j] += ic[j];
            d[512 + lane + 64 * j] += rs[j];
            d[768 + lane + 64 * j] += is[j];
        }
    }
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < EW_SW / 2; ++q) s += red[q][threadIdx.x];
    __syncthreads();
    red[0][threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x >= 256) return;
    const int t = threadIdx.x, er = t >> 4, ecol = t & 15;   // t = row * 16 + column
    const double2 ww = w[(size_t)blockIdx.x * 256 + t];
    const double trc = red[0][t], tic = red[0][256 + t], trs = red[0][512 + t], tis = red[0][768 + t];
    // F+- = w+- (C+- - i S+-),  C+- = rc -+ is,  S+- = ic +- rs
    const double pr = ww.x * (trc - tis), pi = -ww.x * (tic + trs);
    const double mr = ww.y * (trc + tis), mi = -ww.y * (tic - trs);
    const int cg = un.y * 16 + ecol;
    double* f = F + ((size_t)tiles[un.x].x + (cg >> 2)) * 256 + (cg & 3) * 16 + er;
    f[0] = pr + mr;
    f[64] = pi + mi;
    f[128] = pr - mr;
    f[192] = pi - mi;
}

// Potential (and with FIN the force sums) of 16 atoms from every
// EW_PW * splits-th row tile: per tile the product of F with the c phases,
// then one complex product with the row's phase.
// 512 atoms 31 -> 5.5 us and 4,096 atoms (4.4e4 modes) 1,600 -> 98 us against
// a thread per atom with a sine and cosine per (mode, atom); bound by latency
// and by the reads of F, which each 16 atoms make from L2.  A solve of 512
// atoms 2.68 -> 1.17 ms, of 4,096 atoms 57.5 -> 8.9 ms.
template <bool FIN, bool TAB>
__global__ __launch_bounds__(64 * EW_PW) void k_ew_pot(int n, int nrt, EwGeom g, const int4* __restrict__ rows,
                                                       const int2* __restrict__ tiles,
                                                       const double2* __restrict__ tab,
                                                       const double* __restrict__ frac,
                                                       const double* __restrict__ F, double* __restrict__ ypart,
                                                       double* __restrict__ fpart, const int* __restrict__ done) {
    if (done && *done) return;
    __shared__ double red[EW_PW][FIN ? 4 : 1][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int kq = lane >> 4;
    const int i = blockIdx.x * 16 + (lane & 15), ic = min(i, n - 1);
    double y = 0.0, fa = 0.0, fb = 0.0, fc = 0.0;
    for (int rt = blockIdx.y * EW_PW + wv; rt < nrt; rt += EW_PW * gridDim.y) {
        const int2 tl = tiles[rt];   // first K step, K steps in use
        const double* f = F + (size_t)tl.x * 256 + lane;
        ew_d4 gr = {0, 0, 0, 0}, gi = gr, hr = gr, hi = gr;
#pragma unroll 4
        for (int ks = 0; ks < tl.y; ++ks) {
            const double P = f[ks * 256], Q = f[ks * 256 + 64], U = f[ks * 256 + 128], V = f[ks * 256 + 192];
            const int c = min(ks * 4 + kq, g.lim[2]);
            const double2 ec = ew_axis<TAB>(g, tab, frac, n, 2, c, ic);
            gr = ew_mfma(P, ec.x, gr);
            gi = ew_mfma(Q, ec.x, gi);
            gr = ew_mfma(V, -ec.y, gr);
            gi = ew_mfma(U, ec.y, gi);
            if (FIN) {   // the same sums weighted by +-m_c
                const double mc = (double)c;
                hr = ew_mfma(U, mc * ec.x, hr);
                hi = ew_mfma(V, mc * ec.x, hi);
                hr = ew_mfma(Q, -mc * ec.y, hr);
                hi = ew_mfma(P, mc * ec.y, hi);
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int4 row = rows[rt * 16 + kq + 4 * j];
            const double2 e = ew_row<TAB>(g, tab, frac, n, row, ic);
            y += e.x * gr[j] - e.y * gi[j];
            if (FIN) {
                // S cos - C sin = -Im(F e)
                const double im = -(e.x * gi[j] + e.y * gr[j]);
                fa += im * (double)row.x;
                fb += im * (double)row.y;
                fc -= e.x * hi[j] + e.y * hr[j];
            }
        }
    }
    red[wv][0][lane] = y;
    if (FIN) {
        red[wv][1][lane] = fa;
        red[wv][2][lane] = fb;
        red[wv][3][lane] = fc;
    }
    __syncthreads();
    const int q = threadIdx.x >> 4, a = blockIdx.x * 16 + (threadIdx.x & 15);
    if (q >= (FIN ? 4 : 1) || a >= n) return;
    double s = 0.0;
#pragma unroll
    for (int v = 0; v < EW_PW; ++v)
#pragma unroll
        for (int h = 0; h < 4; ++h) s += red[v][q][h * 16 + (threadIdx.x & 15)];
    if (q == 0)
        ypart[(size_t)blockIdx.y * n + a] = s;
    else
        fpart[((size_t)blockIdx.y * n + a) * 3 + q - 1] = s;
}

// yrec[i] = sum of the row splits; with FIN also the forces of the
// reciprocal part, frec_i = -q_i sum k g (added to the pair forces
// afterwards), k = 2 pi H^-1 m.
template <bool FIN>
__global__ void k_ew_sum(int n, int ms, EwGeom g, KParams k, const double* __restrict__ ypart,
                         const double* __restrict__ fpart, const double* __restrict__ src,
                         double* __restrict__ yrec, double* __restrict__ frec, const int* __restrict__ done) {
    if (done && *done) return;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double y = 0.0;
    for (int q = 0; q < ms; ++q) y += ypart[(size_t)q * n + i];
    yrec[i] = y;
    if (FIN) {
        double f[3] = {0.0, 0.0, 0.0};
        for (int q = 0; q < ms; ++q)
            for (int c = 0; c < 3; ++c) f[c] += fpart[((size_t)q * n + i) * 3 + c];
        for (int c = 0; c < 3; ++c)
            frec[3 * i + c] = -src[i] * 2.0 * EW_PI *
                              (k.Hinv[c * 3 + g.ax[0]] * f[0] + k.Hinv[c * 3 + g.ax[1]] * f[1] +
                               k.Hinv[c * 3 + g.ax[2]] * f[2]);
    }
}

__global__ void k_ew_add_forces(int n, const double* __restrict__ frec, double* __restrict__ forces) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < 3 * n) forces[t] += frec[t];
}

template <typename T>
int ew_alloc(T** p, size_t count) {
    if (*p) (void)hipFree(*p);
    *p = nullptr;
    if (hipMalloc((void**)p, sizeof(T) * (count ? count : 1)) != hipSuccess) return QEQ_ENOMEM;
    if (poisonable<T>) debug_poison(*p, sizeof(T) * count);
    return QEQ_OK;
}

}  // namespace

void ew_free(qeq_plan* pl) {
    void* ptrs[] = {pl->ew_lists, pl->ew_w, pl->ew_F, pl->ew_tab, pl->ew_y, pl->ew_f, pl->ew_yrec, pl->ew_frec};
    for (void* q : ptrs)
        if (q) (void)hipFree(q);
    pl->ew_lists = nullptr;
    pl->ew_tab = nullptr;
    pl->ew_w = nullptr;
    pl->ew_F = pl->ew_y = pl->ew_f = pl->ew_yrec = pl->ew_frec = nullptr;
    pl->ew_cap_l = pl->ew_cap_u = pl->ew_cap_t = 0;
    pl->ew_cap_n = 0;
}

// Rows, tiles and units of the current cell, the phase table and the weights;
// buffers grown as needed.
int ew_setup(qeq_plan* pl) {
    const KParams& k = pl->kp;
    const int n = k.n;
    EwGeom& g = pl->ew_geom;
    g = EwGeom{};
    g.kmax2 = 2.0 * log(1e12) / (k.eta * k.eta);
    // multiples of each axis below the cutoff: |m_x| = |k . a_x| / 2 pi
    int lim[3];
    for (int a = 0; a < 3; ++a) {
        const double len = sqrt(k.H[a * 3] * k.H[a * 3] + k.H[a * 3 + 1] * k.H[a * 3 + 1] +
                                k.H[a * 3 + 2] * k.H[a * 3 + 2]);
        lim[a] = (int)ceil(sqrt(g.kmax2) * len / (2.0 * EW_PI)) + 1;
    }
    const int xc = lim[2] >= lim[0] && lim[2] >= lim[1] ? 2 : lim[1] >= lim[0] ? 1 : 0;
    g.ax[0] = xc == 0 ? 1 : 0;
    g.ax[1] = xc == 2 ? 1 : 2;
    g.ax[2] = xc;
    double B[3][3];   // reciprocal vectors of the slots
    for (int x = 0; x < 3; ++x)
        for (int c = 0; c < 3; ++c) B[x][c] = 2.0 * EW_PI * k.Hinv[c * 3 + g.ax[x]];
    const double cc = B[2][0] * B[2][0] + B[2][1] * B[2][1] + B[2][2] * B[2][2];
    auto inside = [&](int a, int b, int c) {
        int m[3];
        m[g.ax[0]] = a;
        m[g.ax[1]] = b;
        m[g.ax[2]] = c;
        double k2 = 0.0;
        for (int q = 0; q < 3; ++q) {
            const double kv =
                2.0 * EW_PI * (k.Hinv[q * 3] * m[0] + k.Hinv[q * 3 + 1] * m[1] + k.Hinv[q * 3 + 2] * m[2]);
            k2 += kv * kv;
        }
        return k2 <= g.kmax2;
    };
    // the m_c inside the cutoff are one interval per (m_a, m_b)
    std::vector<int4> rows;
    long long nm = 0;
    int top = 0;
    for (int a = 0; a <= lim[g.ax[0]]; ++a)
        for (int b = a == 0 ? 0 : -lim[g.ax[1]]; b <= lim[g.ax[1]]; ++b) {
            double d[3], dd = 0.0, dc = 0.0;
            for (int c = 0; c < 3; ++c) {
                d[c] = a * B[0][c] + b * B[1][c];
                dd += d[c] * d[c];
                dc += d[c] * B[2][c];
            }
            const double disc = dc * dc - cc * (dd - g.kmax2);
            if (disc < -1e-9 * cc * g.kmax2) continue;
            const double root = sqrt(std::max(0.0, disc));
            int hi = (int)floor((root - dc) / cc) + 1, lo = (int)ceil((-root - dc) / cc) - 1;
            if (a == 0 && b == 0) lo = 1;
            while (hi >= lo && !inside(a, b, hi)) --hi;
            while (lo <= hi && !inside(a, b, lo)) ++lo;
            if (hi < lo) continue;
            nm += hi - lo + 1;
            if (nm > EW_MAX_MODES) return QEQ_EPLAN;   // cell too large for direct sums
            rows.push_back(make_int4(a, b, std::max(hi, -lo), 0));
            top = std::max(top, std::max(hi, -lo));
        }
    // longest rows first, so that the 16 of a tile are of like length
    std::stable_sort(rows.begin(), rows.end(), [](const int4& p, const int4& q) { return p.z > q.z; });
    const int nrt = ((int)rows.size() + 15) / 16;
    rows.resize((size_t)nrt * 16, make_int4(0, 0, -1, 0));
    std::vector<int2> tiles(nrt), units;
    int ksteps = 0;
    for (int t = 0; t < nrt; ++t) {
        const int len = rows[(size_t)t * 16].z + 1, ct = (len + 15) / 16;
        tiles[t] = make_int2(ksteps, (len + 3) / 4);
        for (int c = 0; c < ct; ++c) units.push_back(make_int2(t, c));
        ksteps += 4 * ct;
    }
    const int nu = (int)units.size();
    g.lim[0] = lim[g.ax[0]];
    g.lim[1] = lim[g.ax[1]];
    g.lim[2] = top;
    g.toff[0] = 0;
    g.toff[1] = g.lim[0] + 1;
    g.toff[2] = g.toff[1] + g.lim[1] + 1;
    g.ntab = g.toff[2] + g.lim[2] + 1;
    pl->ew_nrt = nrt;
    pl->ew_nu = nu;
    // Four waves a block: 1,024 blocks fill every SIMD four deep (256 blocks:
    // 255 us instead of 98 at 4,096 atoms); at least one row tile a wave.
    const int at = (n + 15) / 16;
    pl->ew_ms = std::max(1, std::min({EW_SPLIT_MAX, (EW_BLOCKS + at - 1) / at, (nrt + EW_PW - 1) / EW_PW}));
    const size_t lb = (size_t)nrt * 16 * sizeof(int4) + (size_t)nrt * sizeof(int2) + (size_t)nu * sizeof(int2);
    if (lb > pl->ew_cap_l) {
        pl->ew_cap_l = 0;
        QEQ_TRY(ew_alloc((char**)&pl->ew_lists, lb));
        pl->ew_cap_l = lb;
    }
    if ((size_t)nu > pl->ew_cap_u) {
        pl->ew_cap_u = 0;
        QEQ_TRY(ew_alloc(&pl->ew_w, (size_t)nu * 512));
        QEQ_TRY(ew_alloc(&pl->ew_F, (size_t)nu * 1024));
        pl->ew_cap_u = (size_t)nu;
    }
    if (pl->n_max > pl->ew_cap_n) {
        const size_t nn = (size_t)pl->n_max;
        pl->ew_cap_n = 0;
        QEQ_TRY(ew_alloc(&pl->ew_y, (size_t)EW_SPLIT_MAX * nn));
        QEQ_TRY(ew_alloc(&pl->ew_f, (size_t)EW_SPLIT_MAX * nn * 3));
        QEQ_TRY(ew_alloc(&pl->ew_yrec, nn));
        QEQ_TRY(ew_alloc(&pl->ew_frec, nn * 3));
        pl->ew_cap_n = pl->n_max;
    }
    // Elongated cells with many atoms, whose table would pass 256 MiB (or for
    // which there is no memory), compute each phase where it is used: the same
    // values, no unbounded buffer.  16,384 atoms in a 12 x 12 x 1,800 bohr rod
    // (272 MiB): 1.23 ms a product in place, 0.84 ms with a table, 4.5 ms with
    // a sine and cosine per (mode, atom); a cubic cell passes the line above
    // 50,000 atoms, far beyond where the mesh is the better operator.
    const size_t tb = (size_t)g.ntab * n;
    pl->ew_use_tab = tb * sizeof(double2) <= EW_TABLE_MAX;
    if (pl->ew_use_tab && tb > pl->ew_cap_t) {
        pl->ew_cap_t = 0;
        if (ew_alloc(&pl->ew_tab, tb * 2) == QEQ_OK) {
            pl->ew_cap_t = tb;
        } else {
            (void)hipGetLastError();
            pl->ew_use_tab = false;
        }
    }
    if (nrt == 0) return QEQ_OK;
    std::vector<char> stage(lb);
    const size_t o1 = (size_t)nrt * 16 * sizeof(int4), o2 = o1 + (size_t)nrt * sizeof(int2);
    memcpy(stage.data(), rows.data(), o1);
    memcpy(stage.data() + o1, tiles.data(), (size_t)nrt * sizeof(int2));
    memcpy(stage.data() + o2, units.data(), (size_t)nu * sizeof(int2));
    char* base = (char*)pl->ew_lists;
    pl->ew_rows = (int4*)base;
    pl->ew_tiles = (int2*)(base + o1);
    pl->ew_units = (int2*)(base + o2);
    QEQ_HIP(hipMemcpyAsync(base, stage.data(), lb, hipMemcpyHostToDevice, pl->stream));
    const int nbt = pl->ew_use_tab ? (int)((tb + 255) / 256) : 0;
    hipLaunchKernelGGL(k_ew_tables, dim3(nbt + nu), dim3(256), 0, pl->stream, n, nbt, g, k, pl->frac,
                       (const int4*)pl->ew_rows, (const int2*)pl->ew_units, (double2*)pl->ew_tab,
                       (double2*)pl->ew_w);
    QEQ_HIP(hipGetLastError());
    QEQ_HIP(hipStreamSynchronize(pl->stream));   // the staged lists go out of scope
    return QEQ_OK;
}

namespace {

template <bool TAB>
int ew_rec(qeq_plan* pl, const double* src, const int* done, bool fin) {
    const int n = pl->kp.n, nrt = pl->ew_nrt;
    const EwGeom& g = pl->ew_geom;
    const int4* rows = (const int4*)pl->ew_rows;
    const int2* tiles = (const int2*)pl->ew_tiles;
    const int2* units = (const int2*)pl->ew_units;
    const double2* tab = (const double2*)pl->ew_tab;
    // no reciprocal vector below the cutoff: the sums vanish
    const int ms = nrt > 0 ? pl->ew_ms : 0;
    const dim3 gp((n + 15) / 16, pl->ew_ms);
    if (nrt > 0) {
        hipLaunchKernelGGL(k_ew_sf<TAB>, dim3(pl->ew_nu), dim3(64 * EW_SW), 0, pl->stream, n, g, rows, units, tiles,
                           tab, pl->frac, (const double2*)pl->ew_w, src, pl->ew_F, done);
        if (fin)
            hipLaunchKernelGGL((k_ew_pot<true, TAB>), gp, dim3(64 * EW_PW), 0, pl->stream, n, nrt, g, rows, tiles,
                               tab, pl->frac, pl->ew_F, pl->ew_y, pl->ew_f, done);
        else
            hipLaunchKernelGGL((k_ew_pot<false, TAB>), gp, dim3(64 * EW_PW), 0, pl->stream, n, nrt, g, rows, tiles,
                               tab, pl->frac, pl->ew_F, pl->ew_y, pl->ew_f, done);
    }
    if (fin)
        hipLaunchKernelGGL(k_ew_sum<true>, dim3(nblocks(n)), dim3(QEQ_BLOCK), 0, pl->stream, n, ms, g, pl->kp,
                           pl->ew_y, pl->ew_f, src, pl->ew_yrec, pl->ew_frec, done);
    else
        hipLaunchKernelGGL(k_ew_sum<false>, dim3(nblocks(n)), dim3(QEQ_BLOCK), 0, pl->stream, n, ms, g, pl->kp,
                           pl->ew_y, pl->ew_f, src, pl->ew_yrec, pl->ew_frec, done);
    return qeq_check(hipGetLastError());
}

}  // namespace

// yrec = E_rec src (sorted order); with fin also frec, the reciprocal forces
// (added to the pair forces by launch_ew_forces_add after the final pass).
int launch_ew_rec(qeq_plan* pl, const double* src, const int* done, bool fin) {
    return pl->ew_use_tab ? ew_rec<true>(pl, src, done, fin) : ew_rec<false>(pl, src, done, fin);
}

int launch_ew_forces_add(qeq_plan* pl) {
    const int n = pl->kp.n;
    hipLaunchKernelGGL(k_ew_add_forces, dim3(nblocks(3 * n)), dim3(QEQ_BLOCK), 0, pl->stream, n, pl->ew_frec,
                       pl->fdst);
    return qeq_check(hipGetLastError());
}
