// Batched particle-mesh QEq: many independent periodic structures of uneven
// size, each with its own cell, grid and total charge, solved together.
// Structures are independent (the paper distributes them over ranks for
// training, "Parallelization"); here they advance through the projected CG in
// step, four launches per iteration for the whole batch, each block working on
// one piece of one structure:
//   k_bq_fwd   a few g1 planes: spread, real-to-complex along axis 3, axis 2
//   k_bq_cols  64 lines: axis 1 forward, Green's function, axis 1 inverse
//   k_bq_inv   a few g1 planes: axis 2 and axis 3 inverse, interpolation
//   k_bq_step  a whole structure: pair product, sums, CG update and direction
// Blocks of structures that have converged return at once.  The set-up
// (k_bq_stage, k_bq_pairs, k_bq_green, k_bq_theta, k_bq_self) and the final
// product with energies and forces are shared out the same way.
//
// Why in step and not one workgroup per structure from start to end: a
// structure is then a serial chain on one CU (about 0.45 ms a product), so that
// 48 structures took 20.6 ms on 48 of 256 CUs, and its five separate grid
// passes streamed 170 GB through memory for 1,024 structures (54 ms).  In step,
// a structure's planes and lines spread over the chip, a product moves the half
// spectrum four times (written by fwd, read and written by cols, read by inv)
// instead of eleven, and the real grid stays in LDS.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <vector>

#include "batched_layout.h"
#include "internal.h"

namespace qeqb {

constexpr int BQ_L = 8;         // lanes per atom in the interpolation and pair loops
constexpr int BQ_PAIR_ATOMS = 32;   // atoms of a block of the pair-list kernel
constexpr int BQ_GREEN = 4096;  // Green's function values of a block
static_assert(BQ_MAXP == QEQ_MAXP, "one spline order limit");
constexpr int BQ_OVERFLOW = 100;   // internal status: pair list did not fit

enum { V_Q = 0, V_R, V_P, V_Y, V_DINV, V_CHI, V_DSELF, V_G, V_J, V_SIG, V_CHIRAW };

// Which product the four kernels work on: the starting residual (source q),
// an iteration (source p), the final product (source q, forces).
enum { BQ_INIT = 0, BQ_ITER, BQ_FINAL };

// Per-structure constants prepared on the host.
struct BStruct {
    int n, off, nhalf;          // atoms, first atom, kept half-spectrum points
    int pf, pb;                 // planes of a block of k_bq_fwd and of k_bq_inv
    int km, nm2;                // kept modes: m3 < km, nm2 of the K2 axis-2 ones (|m2| <= (nm2 - 1) / 2, or all)
    int K[3], tw_off[3], bm_off[3];
    int mm[3], nn[3];           // ranges of the C_eta k-space and lattice sums
    double H[9], Hinv[9], M[6];
    double vol, green_pref, bg_pref, q_tot, zeta;
    double rho[3];              // r_cut / perpendicular width, per axis
    long long pcap;             // pairs the slot has room for
    size_t base;                // the slot's byte offset in the scratch buffer
    BSlot slot;
};

// Phases of the per-structure time breakdown (wall-clock ticks, 100 MHz).
enum { PH_SETUP = 0, PH_PAIRS, PH_MESHPREP, PH_SPREAD, PH_FFT, PH_INTERP, PH_VEC, PH_COUNT };

// Per-structure state on the device.
struct BState {
    int status, iters, restarts, q0_rejected;
    int finished;               // results written (or failed)
    int cgdone;                 // the CG of this round has stopped
    int conv;                   // it met the tolerance
    int need_init;              // the residual of q is due
    unsigned long long nnz;     // pairs
    double rz, res, tres, mu, e_qeq, e_elec;
    double chi_sum, dinv_sum, chi_norm, c_eta;
    unsigned long long ticks[PH_COUNT];
};

// Counters the host reads: structures whose CG runs, structures to restart.
struct BCount {
    int running, restarts;
};

struct BArgs {
    int p, self_corr, max_iter;
    double tol, eta, rc2, restart_thr;
    const BStruct* st;
    BState* state;
    BCount* count;
    const float2* tw;
    const float* bmod;
    const double* pos;
    const double* sigma;
    const double* J;
    const double* chi;
    const double* q0;
    double* q_out;
    double* energies;
    double* forces;
    char* scratch;
};

template <typename T>
__device__ __forceinline__ T* slot_ptr(const BArgs& a, const BStruct& S, unsigned off) {
    return reinterpret_cast<T*>(a.scratch + S.base + slot_bytes(off));
}
__device__ __forceinline__ double* slot_vec(const BArgs& a, const BStruct& S, int v) {
    return slot_ptr<double>(a, S, S.slot.vec) + (size_t)v * S.n;
}

__device__ __forceinline__ bool bq_active(const BState& t, int mode) {
    if (t.finished) return false;
    return mode == BQ_INIT ? t.need_init != 0 : mode == BQ_ITER ? t.cgdone == 0 : true;
}

// Adds the block's wall-clock ticks since t0 to a phase of its structure.
__device__ __forceinline__ long long bq_lap(BState& t, int ph, long long t0) {
    const long long now = wall_clock64();
    atomicAdd(&t.ticks[ph], (unsigned long long)(now - t0));
    return now;
}

// Sum of NV doubles over the workgroup, returned to every thread: the waves'
// sums meet in LDS and every thread adds them in the same order.
template <int NV>
__device__ __forceinline__ void wg_sum(double* v) {
    __shared__ double red[16][NV];
    const int nw = (blockDim.x + 63) >> 6;
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = wave_sum(v[k]);
    __syncthreads();   // earlier readers of red
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) red[threadIdx.x >> 6][k] = v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        double s = red[0][k];
        for (int w = 1; w < nw; ++w) s += red[w][k];
        v[k] = s;
    }
}

// ------------------------------------------------------------------ set-up
// One block per structure: validation, fractional coordinates, atoms sorted by
// their home plane h1 (ties by index, so that every later sum has one order),
// spline weights, diagonal, starting charges, norms and the reciprocal self
// constant
//   C_eta = (4 pi / V) sum_{k != 0} exp(-eta^2 k^2 / 2) / k^2
// by a second split of width zeta: k-space sum with zeta plus the lattice sum
// of the difference kernel, minus 2 pi (zeta^2 - eta^2) / V.
__global__ __launch_bounds__(1024) void k_bq_stage(BArgs a, const int* __restrict__ order) {
    const int s = order[blockIdx.x];
    const BStruct& S = a.st[s];
    BState& T = a.state[s];
    const int n = S.n, p = a.p, tid = threadIdx.x;
    const double Q = S.q_tot;
    const long long t0 = wall_clock64();
    __shared__ int err, key[1024], hcnt[BQ_KAX + 1];
    if (tid == 0) err = 0;
    if (tid <= BQ_KAX) hcnt[tid] = 0;
    __syncthreads();
    const bool live = tid < n;
    const int o = S.off + tid;
    double x[3] = {0.0, 0.0, 0.0}, fr[3] = {0.0, 0.0, 0.0}, sg = 1.0, jj = 1.0, ch = 0.0, q = 0.0;
    int h[3] = {0, 0, 0};
    if (live) {
        for (int c = 0; c < 3; ++c) x[c] = a.pos[3 * (size_t)o + c];
        sg = a.sigma[o];
        jj = a.J[o];
        ch = a.chi[o];
        q = a.q0 ? a.q0[o] : Q / (double)n;
        if (!isfinite(q)) q = Q / (double)n;
        const bool ok = isfinite(x[0]) && isfinite(x[1]) && isfinite(x[2]) && isfinite(ch) && sg > 0.0 && jj > 0.0 &&
                        isfinite(sg) && isfinite(jj);
        if (!ok) err = 1;
        for (int c = 0; c < 3; ++c) {
            double v = x[0] * S.Hinv[0 * 3 + c] + x[1] * S.Hinv[1 * 3 + c] + x[2] * S.Hinv[2 * 3 + c];
            v -= floor(v);
            if (!(v >= 0.0 && v < 1.0)) v = 0.0;
            fr[c] = v;
            const int K = S.K[c];
            int g = (int)floor(v * (double)K);
            h[c] = g < 0 ? 0 : (g >= K ? K - 1 : g);
        }
        key[tid] = h[0];
        atomicAdd(&hcnt[h[0]], 1);
    }
    __syncthreads();
    if (err) {
        if (tid == 0) {
            T.status = QEQ_EINVAL;
            T.finished = 1;
            atomicSub(&a.count->running, 1);
        }
        return;
    }
    int* hs = slot_ptr<int>(a, S, S.slot.hstart);
    if (tid == 0) {
        int run = 0;
        for (int b = 0; b < S.K[0]; ++b) {
            const int c = hcnt[b];
            hs[b] = run;
            hcnt[b] = run;
            run += c;
        }
        hs[S.K[0]] = run;
    }
    __syncthreads();
    double acc[3] = {0.0, 0.0, 0.0};
    int at = 0;
    double ce = 0.0;
    if (live) {
        at = hcnt[h[0]];
        for (int t = 0; t < tid; ++t) at += key[t] == h[0] ? 1 : 0;
        slot_ptr<int>(a, S, S.slot.perm)[at] = tid;
        float* wts = slot_ptr<float>(a, S, S.slot.wts) + (size_t)at * 3 * QEQ_MAXP;
        float* dwts = slot_ptr<float>(a, S, S.slot.dwts) + (size_t)at * 3 * QEQ_MAXP;
        double* frac = slot_ptr<double>(a, S, S.slot.frac);
        int* home = slot_ptr<int>(a, S, S.slot.home);
        for (int c = 0; c < 3; ++c) {
            frac[3 * at + c] = fr[c];
            home[4 * at + c] = h[c];
            double w[QEQ_MAXP], dw[QEQ_MAXP];
            bspline_weights<double>(fr[c] * (double)S.K[c] - (double)h[c], p, w, dw);
            for (int k = 0; k < QEQ_MAXP; ++k) {
                wts[c * QEQ_MAXP + k] = k < p ? (float)w[k] : 0.f;
                dwts[c * QEQ_MAXP + k] = k < p ? (float)dw[k] : 0.f;
            }
        }
        const double rsqpi = 0.56418958354775628695;
        ce = ch + S.bg_pref * Q * sg * sg;
        slot_vec(a, S, V_CHI)[at] = ce;
        slot_vec(a, S, V_CHIRAW)[at] = ch;
        slot_vec(a, S, V_SIG)[at] = sg;
        slot_vec(a, S, V_J)[at] = jj;
        slot_vec(a, S, V_DSELF)[at] = rsqpi / sg - 0.79788456080286535588 / a.eta;
        const double di = 1.0 / (jj + rsqpi / sg);
        slot_vec(a, S, V_DINV)[at] = di;
        acc[0] = ce;
        acc[1] = di;
        acc[2] = q;
    }
    wg_sum<3>(acc);
    const double chi_sum = acc[0], dinv_sum = acc[1];
    if (live) slot_vec(a, S, V_Q)[at] = q + (Q - acc[2]) / (double)n;
    // norm of the projected right-hand side and the two sums of C_eta
    double v[3] = {0.0, 0.0, 0.0};
    if (live) {
        const double d = ce - chi_sum / (double)n;
        v[0] = d * d;
    }
    {
        const double X = 6.5 * 1.41421356237309504880;
        const double zeta = S.zeta, eta = a.eta;
        const double kmax = X / zeta, rmax = X * zeta;
        const int w1 = 2 * S.mm[0] + 1, w2 = 2 * S.mm[1] + 1, w3 = 2 * S.mm[2] + 1;
        for (int t = tid; t < w1 * w2 * w3; t += 1024) {
            const int m3 = t % w3 - S.mm[2], m2 = (t / w3) % w2 - S.mm[1], m1 = t / (w3 * w2) - S.mm[0];
            if (!m1 && !m2 && !m3) continue;
            double k[3];
            for (int c = 0; c < 3; ++c)
                k[c] = 6.283185307179586477 * (S.Hinv[c * 3 + 0] * m1 + S.Hinv[c * 3 + 1] * m2 + S.Hinv[c * 3 + 2] * m3);
            const double k2 = k[0] * k[0] + k[1] * k[1] + k[2] * k[2];
            if (k2 > kmax * kmax) continue;
            v[1] += exp(-0.5 * zeta * zeta * k2) / k2;
        }
        const int v1 = 2 * S.nn[0] + 1, v2 = 2 * S.nn[1] + 1, v3 = 2 * S.nn[2] + 1;
        const double s2 = 0.70710678118654752440;
        for (int t = tid; t < v1 * v2 * v3; t += 1024) {
            const int n3 = t % v3 - S.nn[2], n2 = (t / v3) % v2 - S.nn[1], n1 = t / (v3 * v2) - S.nn[0];
            double y[3];
            for (int c = 0; c < 3; ++c) y[c] = n1 * S.H[0 * 3 + c] + n2 * S.H[1 * 3 + c] + n3 * S.H[2 * 3 + c];
            const double r = sqrt(y[0] * y[0] + y[1] * y[1] + y[2] * y[2]);
            if (r > rmax) continue;
            v[2] += r < 1e-12 ? 0.79788456080286535588 * (1.0 / eta - 1.0 / zeta)
                              : (erf(r * s2 / eta) - erf(r * s2 / zeta)) / r;
        }
    }
    wg_sum<3>(v);
    if (tid == 0) {
        const double pi = 3.14159265358979323846;
        T.chi_sum = chi_sum;
        T.dinv_sum = dinv_sum;
        T.chi_norm = sqrt(v[0]);
        T.c_eta = v[1] * 4.0 * pi / S.vol + v[2] - 2.0 * pi * (S.zeta * S.zeta - a.eta * a.eta) / S.vol;
        T.need_init = 1;
        bq_lap(T, PH_SETUP, t0);
    }
}

// Images n of the pair (i, j) with |x_a + n_a| <= rho_a on every axis, where
// x = s_j - s_i is wrapped to [-1/2, 1/2], and |r_j + n H - r_i| < r_cut.
// EMIT writes j, r_i - r_j(image) and, in the places of K'/r and K, the two
// halves of the FP64 distance.
template <bool EMIT>
__device__ __forceinline__ int bq_pair_images(const BStruct& S, const double* si, const double* sj, bool same,
                                              double rc2, int j, int* col, float* kval, float4* pdr, long long at,
                                              long long cap) {
    double x[3];
    int lo[3], hi[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double d = sj[a] - si[a];
        d -= rint(d);
        x[a] = d;
        lo[a] = (int)ceil(-S.rho[a] - d);
        hi[a] = (int)floor(S.rho[a] - d);
    }
    int c = 0;
    for (int n1 = lo[0]; n1 <= hi[0]; ++n1)
        for (int n2 = lo[1]; n2 <= hi[1]; ++n2)
            for (int n3 = lo[2]; n3 <= hi[2]; ++n3) {
                if (same && n1 == 0 && n2 == 0 && n3 == 0) continue;
                const double f0 = x[0] + n1, f1 = x[1] + n2, f2 = x[2] + n3;
                const double dx = f0 * S.H[0] + f1 * S.H[3] + f2 * S.H[6];
                const double dy = f0 * S.H[1] + f1 * S.H[4] + f2 * S.H[7];
                const double dz = f0 * S.H[2] + f1 * S.H[5] + f2 * S.H[8];
                const double r2 = dx * dx + dy * dy + dz * dz;
                if (r2 >= rc2) continue;
                if (EMIT && at + c < cap) {
                    const double rr = sqrt(r2);
                    col[at + c] = j;
                    kval[at + c] = __int_as_float(__double2loint(rr));
                    pdr[at + c] =
                        make_float4((float)(-dx), (float)(-dy), (float)(-dz), __int_as_float(__double2hiint(rr)));
                }
                ++c;
            }
    return c;
}

// Pair list of 32 atoms: count, one reservation of the block's rows in the
// structure's list, fill (8 lanes per atom, in j order; where a row starts
// does not matter to any sum).  Past the capacity only the count goes on.
// The fill writes distances and a second pass over the row turns them into
// kernel values: about one candidate in four is a pair, and the error functions
// inside the fill ran for a whole wave wherever one lane had one (1,024
// structures 1.50 -> 1.09 ms, 48 structures 132 -> 107 us).
__global__ __launch_bounds__(256) void k_bq_pairs(BArgs a, const int2* __restrict__ units) {
    const int2 u = units[blockIdx.x];
    const BStruct& S = a.st[u.x];
    BState& T = a.state[u.x];
    if (T.finished) return;
    const long long t0 = wall_clock64();
    const int n = S.n, tid = threadIdx.x;
    __shared__ double fr[3 * 1024], sgs[1024];
    __shared__ int cnt[BQ_PAIR_ATOMS];
    __shared__ long long rowat[BQ_PAIR_ATOMS];
    const double* frac = slot_ptr<double>(a, S, S.slot.frac);
    const double* sig = slot_vec(a, S, V_SIG);
    for (int t = tid; t < 3 * n; t += 256) fr[t] = frac[t];
    for (int t = tid; t < n; t += 256) sgs[t] = sig[t];
    __syncthreads();
    const int l = tid & (BQ_L - 1), r = tid / BQ_L;
    const int i = u.y * BQ_PAIR_ATOMS + r;
    double si[3] = {0.0, 0.0, 0.0};
    int c = 0;
    if (i < n) {
        for (int t = 0; t < 3; ++t) si[t] = fr[3 * i + t];
        for (int j = l; j < n; j += BQ_L)
            c += bq_pair_images<false>(S, si, fr + 3 * j, i == j, a.rc2, j, nullptr, nullptr, nullptr, 0, 0);
    }
#pragma unroll
    for (int off = BQ_L / 2; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
    if (l == 0) cnt[r] = c;
    __syncthreads();
    if (tid == 0) {
        int tot = 0;
        for (int t = 0; t < BQ_PAIR_ATOMS; ++t) tot += cnt[t];
        long long at = (long long)atomicAdd(&T.nnz, (unsigned long long)tot);
        for (int t = 0; t < BQ_PAIR_ATOMS; ++t) {
            rowat[t] = at;
            at += cnt[t];
        }
    }
    __syncthreads();
    int* col = slot_ptr<int>(a, S, S.slot.col);
    float* kval = slot_ptr<float>(a, S, S.slot.kval);
    float4* pdr = slot_ptr<float4>(a, S, S.slot.pdr);
    if (i < n) {
        long long cursor = rowat[r];
        if (l == 0) {
            int2* row = slot_ptr<int2>(a, S, S.slot.row);
            // rows past the capacity are never read (the structure goes again)
            row[i] = cursor + c <= S.pcap ? make_int2((int)cursor, (int)cursor + c) : make_int2(0, 0);
        }
        for (int jb = 0; jb < n; jb += BQ_L) {
            const int j = jb + l;
            int k = 0;
            if (j < n)
                k = bq_pair_images<false>(S, si, fr + 3 * j, i == j, a.rc2, j, nullptr, nullptr, nullptr, 0, 0);
            int incl = k;
#pragma unroll
            for (int d = 1; d < BQ_L; d <<= 1) {
                const int y = __shfl_up(incl, d, BQ_L);
                if (l >= d) incl += y;
            }
            const int total = __shfl(incl, BQ_L - 1, BQ_L);
            if (k)
                bq_pair_images<true>(S, si, fr + 3 * j, i == j, a.rc2, j, col, kval, pdr, cursor + incl - k, S.pcap);
            cursor += total;
        }
    }
    __syncthreads();   // the rows' entries, written by other lanes
    if (i < n) {
        const double sgi = sgs[i];
        const long long e1 = min(rowat[r] + cnt[r], S.pcap);
        for (long long e = rowat[r] + l; e < e1; e += BQ_L) {
            const float hi = pdr[e].w, lo = kval[e];
            const double sj = sgs[col[e]];
            double K, dKr;
            pair_kernel(__hiloint2double(__float_as_int(hi), __float_as_int(lo)), sqrt(sgi * sgi + sj * sj), a.eta, &K,
                        &dKr);
            kval[e] = (float)K;
            pdr[e].w = (float)dKr;
        }
    }
    if (tid == 0) bq_lap(T, PH_PAIRS, t0);
}

// Green's function of the split times the B-spline moduli (SI "Ewald
// Summation" Gaussian filter, eq. matvec 4 pi / k^2) on the half spectrum
// (m3 <= K3 / 2): zero at m = 0 and on the Nyquist planes, as in the
// single-structure path.
__device__ __forceinline__ float bq_green(const BStruct& S, double eta, int m1, int m2, int m3, const float* b1,
                                          const float* b2, const float* b3) {
    const int K1 = S.K[0], K2 = S.K[1], K3 = S.K[2];
    if ((m1 | m2 | m3) == 0) return 0.f;
    if (2 * m1 == K1 || 2 * m2 == K2 || 2 * m3 == K3) return 0.f;
    const double x1 = m1 <= K1 / 2 ? m1 : m1 - K1;
    const double x2 = m2 <= K2 / 2 ? m2 : m2 - K2;
    const double x3 = m3;
    const double q = S.M[0] * x1 * x1 + S.M[1] * x2 * x2 + S.M[2] * x3 * x3 +
                     2.0 * (S.M[3] * x1 * x2 + S.M[4] * x1 * x3 + S.M[5] * x2 * x3);
    const double k2 = 39.478417604357434475 * q;   // (2 pi)^2
    const double g = S.green_pref * exp(-0.5 * eta * eta * k2) / k2;
    return (float)g * b1[m1] * b2[m2] * b3[m3];
}

__global__ __launch_bounds__(256) void k_bq_green(BArgs a, const int2* __restrict__ units) {
    const int2 u = units[blockIdx.x];
    const BStruct& S = a.st[u.x];
    BState& T = a.state[u.x];
    if (T.finished) return;
    const long long t0 = wall_clock64();
    float* G = slot_ptr<float>(a, S, S.slot.G);
    const int nm2 = S.nm2, K3h = S.km;
    const float *b1 = a.bmod + S.bm_off[0], *b2 = a.bmod + S.bm_off[1], *b3 = a.bmod + S.bm_off[2];
    const int end = min(S.nhalf, (u.y + 1) * BQ_GREEN);
    for (int t = u.y * BQ_GREEN + threadIdx.x; t < end; t += 256) {
        const int m3 = t % K3h, r = t / K3h;
        G[t] = bq_green(S, a.eta, r / nm2, bq_m2(r % nm2, nm2, S.K[1]), m3, b1, b2, b3);
    }
    if (threadIdx.x == 0) bq_lap(T, PH_MESHPREP, t0);
}

// ------------------------------------------------------------------ mesh
// Layout in the slot: half spectrum C[g1][e][m3] of the kept modes (m3
// contiguous, below km; e counts the kept m2), the Green's function G in the
// same layout: modes with exp(-eta^2 k^2 / 2) below 2^-30 are left out as in
// the single-structure passes (64% of the modes stay at 0.8 bohr and eta = 2).
// Every axis length of the batched path has a compile-time transform.
#define BQ_FOR_EACH_LEN(X) X(12) X(16) X(20) X(24) X(32) X(36) X(40) X(48) X(60) X(64)

template <bool INV>
__device__ __forceinline__ void bq_fft_axis2(float2* X2, int K2, const float2* tw, int tid) {
    switch (K2) {
#define X(KK) case KK: fft_ct<KK, BQ_NC2, BQ_KS2, BQ_NT, INV>(X2, tw, tid); break;
        BQ_FOR_EACH_LEN(X)
#undef X
    }
}

template <bool INV>
__device__ __forceinline__ void bq_fft_lines(float2* buf, int K, const float2* tw, int tid) {
    switch (K) {
#define X(KK) case KK: fft_ct<KK, BQ_NC, BQ_KS, BQ_NT, INV>(buf, tw, tid); break;
        BQ_FOR_EACH_LEN(X)
#undef X
    }
}

// The atoms that reach each of a block's planes: those with home planes g1 ..
// g1 + p - 1, one (wrapped) index range per plane.  first / cnt in LDS, off =
// their running total.
__device__ __forceinline__ void bq_ranges(const int* hs, int K1, int n, int p, int g1a, int planes, int tid, int* first,
                                          int* off) {
    if (tid < planes) {
        const int g = g1a + tid, e = g + p;
        first[tid] = hs[g];
        off[tid + 1] = e <= K1 ? hs[e] - hs[g] : n - hs[g] + hs[e - K1];
    }
    __syncthreads();
    if (tid == 0) {
        off[0] = 0;
        for (int j = 0; j < planes; ++j) off[j + 1] += off[j];
    }
    __syncthreads();
}

// A 64-bit sum below 2^51 as FP32, rounded once: exact in FP64 (the conversion
// that hipcc expands for 64-bit integers takes three times the instructions).
__device__ __forceinline__ float bq_float(long long x) {
    return (float)fma((double)(int)(x >> 32), 4294967296.0, (double)(unsigned)x);
}

// Spread, real-to-complex along axis 3 and axis 2 forward of a block's planes.
// The spread accumulates in 64-bit fixed point with integer LDS atomics (exact,
// order-independent; FP32 LDS atomics are several times slower on gfx950),
// scaled per block so that no sum can overflow: a grid value is a sum over the
// block's candidate atoms of src times a weight product <= 1, each candidate at
// most once, so |value| <= sum |src| < 2^e and the scale is 2^(50 - e); each
// term is rounded to an integer by one FP64 fused multiply-add with 1.5 * 2^52
// (its bit pattern minus the constant's is the integer, exact below 2^51).
// Planes of a block: as many as fill 128 real rows (64 complex lines of two)
// and 56 half-spectrum columns, so that its barriers pass with several planes'
// work behind them, and whose accumulator takes at most 38,400 bytes, so that
// four blocks share a CU: the block waits at its barriers, not for the VALU (58
// KB, two blocks a CU: 226 us a launch for 1,024 structures, 18.1 for 48; now
// 172 and 15.4.  Accumulating the planes in two halves instead kept the wide
// blocks but took 95 registers: 272 us).
__global__ __launch_bounds__(BQ_NT) void k_bq_fwd(BArgs a, const int2* __restrict__ units, int mode) {
    extern __shared__ float2 lds[];
    const int2 u = units[blockIdx.x];
    if (u.x < 0) return;
    const BStruct& S = a.st[u.x];
    BState& T = a.state[u.x];
    if (!bq_active(T, mode)) return;
    long long t0 = wall_clock64();
    __shared__ float2 tw3[BQ_KAX], tw2[BQ_KAX];
    __shared__ int first[BQ_PB], off[BQ_PB + 1];
    const int tid = threadIdx.x, n = S.n, p = a.p;
    const int K1 = S.K[0], K2 = S.K[1], K3 = S.K[2], km = S.km;
    const int g1a = u.y * S.pf, planes = min(S.pf, K1 - g1a);
    const int RW = S.pf * K2;                                // accumulator rows
    long long* acc = reinterpret_cast<long long*>(lds);      // [K3][RW]
    unsigned long long* acc_u = reinterpret_cast<unsigned long long*>(lds);
    float2* buf = lds;                                       // [K3][BQ_KS], in its place
    float2* X2 = lds;                                        // [K2][BQ_KS2], in its place again
    const double* src = slot_vec(a, S, mode == BQ_ITER ? V_P : V_Q);
    const int* home = slot_ptr<int>(a, S, S.slot.home);
    const float* wts = slot_ptr<float>(a, S, S.slot.wts);
    const int* hs = slot_ptr<int>(a, S, S.slot.hstart);
    if (tid < K3) tw3[tid] = a.tw[S.tw_off[2] + tid];
    if (tid >= BQ_KAX && tid - BQ_KAX < K2) tw2[tid - BQ_KAX] = a.tw[S.tw_off[1] + tid - BQ_KAX];
    for (int t = tid; t < K3 * RW / 2; t += BQ_NT) reinterpret_cast<int4*>(acc)[t] = make_int4(0, 0, 0, 0);
    // all candidates of the block: home planes g1a .. g1a + planes + p - 2
    const int e = g1a + planes + p - 1;
    const int c0 = hs[g1a], ncand = e <= K1 ? hs[e] - c0 : n - c0 + hs[e - K1];
    bq_ranges(hs, K1, n, p, g1a, planes, tid, first, off);
    double v[1] = {0.0};
    for (int c = tid; c < ncand; c += BQ_NT) {
        const int i = c0 + c;
        v[0] += fabs(src[i < n ? i : i - n]);
    }
    wg_sum<1>(v);   // its barriers also order the clears above
    int ex = 0;
    (void)frexp(v[0] > 0.0 ? v[0] : 1.0, &ex);
    const float scale = ldexpf(1.0f, max(-126, min(126, 50 - ex)));
    constexpr double RND = 6755399441055744.0;   // 1.5 * 2^52
    // two lanes per (atom, plane), half of the axis-2 rows each: a row's set-up
    // is shared by p terms and an item's by p^2 / 2 (eight lanes with one row
    // each took 2.4 times the instructions)
    {
        const int items = off[planes], hp = p >> 1, k20 = (tid & 1) * hp;
        for (int t = tid >> 1; t < items; t += BQ_NT / 2) {
            int j = 0;
            while (t >= off[j + 1]) ++j;
            int i = first[j] + (t - off[j]);
            if (i >= n) i -= n;
            const int4 hm = *reinterpret_cast<const int4*>(home + 4 * i);
            int k1 = hm.x - (g1a + j);
            if (k1 < 0) k1 += K1;
            const float* w = wts + (size_t)i * 3 * QEQ_MAXP;
            const float a1 = (float)src[i] * w[k1];
            const float4 wa = *reinterpret_cast<const float4*>(w + 2 * QEQ_MAXP);
            const float4 wb = *reinterpret_cast<const float4*>(w + 2 * QEQ_MAXP + 4);
            const double w3[8] = {wa.x, wa.y, wa.z, wa.w, wb.x, wb.y, wb.z, wb.w};
            int g2 = hm.y - k20;
            if (g2 < 0) g2 += K2;
            unsigned long long* col[QEQ_MAXP];
#pragma unroll
            for (int k3 = 0; k3 < QEQ_MAXP; ++k3) {
                int g3 = hm.z - k3;
                if (g3 < 0) g3 += K3;
                col[k3] = acc_u + g3 * RW + j * K2;
            }
            for (int q = 0; q < hp; ++q) {
                const double a0 = (double)(a1 * w[QEQ_MAXP + k20 + q] * scale);
#pragma unroll
                for (int k3 = 0; k3 < QEQ_MAXP; ++k3) {
                    if (k3 >= p) break;
                    const long long b = __double_as_longlong(fma(a0, w3[k3], RND));
                    const unsigned hi = (unsigned)(b >> 32) - 0x43380000u;
                    atomicAdd(col[k3] + g2, ((unsigned long long)hi << 32) | (unsigned)b);
                }
                g2 = g2 == 0 ? K2 - 1 : g2 - 1;
            }
        }
    }
    __syncthreads();
    if (tid == 0) t0 = bq_lap(T, PH_SPREAD, t0);
    // fixed point -> FP32 complex lines (rows 2 c and 2 c + 1), through registers
    {
        const float inv = 1.0f / scale;
        constexpr int PER = (BQ_KAX * BQ_NC + BQ_NT - 1) / BQ_NT;
        const int half = RW >> 1;
        float2 z[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int t = tid + q * BQ_NT, g3 = t / BQ_NC, c = t % BQ_NC;
            z[q] = make_float2(0.f, 0.f);
            if (g3 < K3 && c < half) {
                const longlong2 x = *reinterpret_cast<const longlong2*>(acc + g3 * RW + 2 * c);
                z[q] = make_float2(bq_float(x.x) * inv, bq_float(x.y) * inv);
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int t = tid + q * BQ_NT, g3 = t / BQ_NC, c = t % BQ_NC;
            if (g3 < K3) buf[g3 * BQ_KS + c] = z[q];
        }
        __syncthreads();
    }
    bq_fft_lines<false>(buf, K3, tw3, tid);
    // the two rows' half spectra: X2[g2][j km + m3], a thread keeps its row
    const int rows = planes * K2;
    {
        const int r = tid & (2 * BQ_NC - 1);
        const int j = r / K2, g2 = r - j * K2;
        const float2* line = buf + (r >> 1);
        float2* x = X2 + g2 * BQ_KS2 + j * km;
        constexpr int STEP = BQ_NT / (2 * BQ_NC), PM = (BQ_KAX / 2 + STEP) / STEP;
        const int mf = tid / (2 * BQ_NC);
        float2 xv[PM];
#pragma unroll
        for (int q = 0; q < PM; ++q) {
            const int m = mf + q * STEP;
            if (m < km) {
                const float2 Z = line[m * BQ_KS];
                float2 Zc = line[(m == 0 ? 0 : K3 - m) * BQ_KS];
                Zc.y = -Zc.y;
                const float2 d = csub(Z, Zc);
                const float2 ev = make_float2(0.5f * (Z.x + Zc.x), 0.5f * (Z.y + Zc.y));
                const float2 od = make_float2(0.5f * d.y, -0.5f * d.x);
                xv[q] = (r & 1) ? od : ev;
            }
        }
        __syncthreads();
        if (r < rows) {
#pragma unroll
            for (int q = 0; q < PM; ++q) {
                const int m = mf + q * STEP;
                if (m < km) x[m] = xv[q];
            }
        }
    }
    __syncthreads();
    bq_fft_axis2<false>(X2, K2, tw2, tid);
    float2* C = slot_ptr<float2>(a, S, S.slot.C) + (size_t)g1a * S.nm2 * km;
    const int kept = planes * S.nm2;
    for (BqWalk w(tid, S.nm2, km, K2); w.row < kept; w.next())
        for (int m = tid & 31; m < km; m += 32) C[w.row * km + m] = X2[w.at() + m];
    if (tid == 0) bq_lap(T, PH_FFT, t0);
}

// Real-space pair product of 64 atoms, eight lanes per atom: V_Y[i] = sum_j K_ij
// src_j; for the final product also fpair[i] = sum_j K'_ij / r_ij src_j (r_i - r_j).
// It needs nothing of the mesh, so its blocks ride with the axis-1 lines, the
// lightest of the product's launches (in k_bq_step, one block per structure, it
// took two thirds of that kernel's 17 us for 512 atoms).
__device__ __forceinline__ void bq_pair_product(const BArgs& a, const BStruct& S, int chunk, int mode) {
    const int tid = threadIdx.x, n = S.n;
    const int l = tid & (BQ_L - 1), i = chunk * (BQ_NT / BQ_L) + tid / BQ_L;
    const bool fin = mode == BQ_FINAL;
    const double* src = slot_vec(a, S, mode == BQ_ITER ? V_P : V_Q);
    const int* col = slot_ptr<int>(a, S, S.slot.col);
    const float* kval = slot_ptr<float>(a, S, S.slot.kval);
    const float4* pdr = slot_ptr<float4>(a, S, S.slot.pdr);
    double v = 0.0, f[3] = {0.0, 0.0, 0.0};
    if (i < n) {
        const int2 row = slot_ptr<int2>(a, S, S.slot.row)[i];
        for (int e0 = row.x + l; e0 < row.y; e0 += 4 * BQ_L) {
            int cj[4];
            float kv[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int e = e0 + q * BQ_L;
                cj[q] = e < row.y ? col[e] : 0;
                kv[q] = e < row.y ? kval[e] : 0.f;
            }
            double vj[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) vj[q] = src[cj[q]];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                v += (double)kv[q] * vj[q];
                if (fin && e0 + q * BQ_L < row.y) {
                    const float4 d = pdr[e0 + q * BQ_L];
                    const double c = (double)d.w * vj[q];
                    f[0] += c * d.x;
                    f[1] += c * d.y;
                    f[2] += c * d.z;
                }
            }
        }
    }
#pragma unroll
    for (int d = BQ_L / 2; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
    if (fin) {
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int d = BQ_L / 2; d > 0; d >>= 1) f[c] += __shfl_xor(f[c], d, 64);
    }
    if (i < n && l == 0) {
        slot_vec(a, S, V_Y)[i] = v;
        if (fin) {
            double* fp = slot_ptr<double>(a, S, S.slot.fpair);
            for (int c = 0; c < 3; ++c) fp[3 * i + c] = f[c];
        }
    }
}

// 64 lines (m2, m3) along axis 1: forward, times G, inverse, in place; with
// THETA the inverse of G alone (the mesh kernel around the origin).  A line's
// elements and Green's function values are requested before the first LDS
// store, so a block costs one memory round trip.  Units with a negative piece
// -1 - c: the pair product of atoms 64 c ...
template <bool THETA>
__global__ __launch_bounds__(BQ_NT) void k_bq_cols(BArgs a, const int2* __restrict__ units, int mode) {
    extern __shared__ float2 lds[];
    const int2 u = units[blockIdx.x];
    if (u.x < 0) return;
    const BStruct& S = a.st[u.x];
    BState& T = a.state[u.x];
    if (!bq_active(T, mode)) return;
    const long long t0 = wall_clock64();
    if (!THETA && u.y < 0) {
        // (a pair list that did not fit is never read: the structure goes again)
        if ((long long)T.nnz <= S.pcap) bq_pair_product(a, S, -1 - u.y, mode);
        if (threadIdx.x == 0) bq_lap(T, PH_INTERP, t0);
        return;
    }
    __shared__ float2 tw1[BQ_KAX];
    const int tid = threadIdx.x;
    const int K1 = S.K[0];
    const int nl = S.nm2 * S.km;
    const int c = tid % BQ_NC, k0 = tid / BQ_NC;
    const int L = u.y * BQ_NC + c;
    const bool live = L < nl;
    constexpr int KSTEP = BQ_NT / BQ_NC, MAXIT = BQ_KAX / KSTEP;
    float2* C = slot_ptr<float2>(a, S, S.slot.C);
    const float* G = slot_ptr<float>(a, S, S.slot.G);
    if (tid < K1) tw1[tid] = a.tw[S.tw_off[0] + tid];
    float gv[MAXIT];
    float2 v[MAXIT];
#pragma unroll
    for (int q = 0; q < MAXIT; ++q) {
        const int k = k0 + q * KSTEP;
        gv[q] = 0.f;
        v[q] = make_float2(0.f, 0.f);
        if (k < K1 && live) {
            gv[q] = G[(size_t)k * nl + L];
            if (!THETA) v[q] = C[(size_t)k * nl + L];
        }
    }
#pragma unroll
    for (int q = 0; q < MAXIT; ++q) {
        const int k = k0 + q * KSTEP;
        if (k < K1) lds[k * BQ_KS + c] = THETA ? make_float2(gv[q], 0.f) : v[q];
    }
    __syncthreads();
    if (!THETA) {
        bq_fft_lines<false>(lds, K1, tw1, tid);
#pragma unroll
        for (int q = 0; q < MAXIT; ++q) {
            const int k = k0 + q * KSTEP;
            if (k < K1) lds[k * BQ_KS + c] = cscale(lds[k * BQ_KS + c], gv[q]);
        }
        __syncthreads();
    }
    bq_fft_lines<true>(lds, K1, tw1, tid);
    if (live)
        for (int k = k0; k < K1; k += KSTEP) C[(size_t)k * nl + L] = lds[k * BQ_KS + c];
    if (tid == 0) bq_lap(T, THETA ? PH_MESHPREP : PH_FFT, t0);
}

// Axis 2 and axis 3 inverse of `planes` planes from g1a: the potential of row
// r = j K2 + g2 at g3 is bf[2 (g3 BQ_KS + (r >> 1)) + (r & 1)].  Two rows a, b
// of half spectra form Z(m) = X_a(m) + i X_b(m) over the full axis (Hermitian
// extension); the inverse transform returns row a in the real and row b in the
// imaginary part.  buf [K3][BQ_KS] and X2 [K2][BQ_KS2] share their place: 33 KB at
// most, so that four blocks share a CU (two with both side by side:
// 228 -> 147 us a launch for 1,024 structures).
__device__ __forceinline__ void bq_inverse_planes(const BArgs& a, const BStruct& S, int g1a, int planes, float2* buf,
                                              const float2* tw2, const float2* tw3, int tid) {
    const int K2 = S.K[1], K3 = S.K[2], km = S.km;
    float2* X2 = buf;   // the packed lines take its place through registers
    const float2* C = slot_ptr<float2>(a, S, S.slot.C) + (size_t)g1a * S.nm2 * km;
    const int rows = planes * K2, cols = planes * km, kept = planes * S.nm2;
    // every load of the thread first, then the LDS stores
    constexpr int PER = 2 * BQ_NC / BqWalk::ROWS;
    float2 v[PER], ve[PER];
    const int m0 = tid & 31;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int row = (tid >> 5) + q * BqWalk::ROWS;
        if (row < kept && m0 < km) v[q] = C[row * km + m0];
        if (row < kept && m0 + 32 < km) ve[q] = C[row * km + m0 + 32];
    }
    BqWalk w(tid, S.nm2, km, K2);
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        if (w.row < kept) {
            float2* x = X2 + w.at();
            if (m0 < km) x[m0] = v[q];
            if (m0 + 32 < km) x[m0 + 32] = ve[q];
        }
        w.next();
    }
    // the rows of m2 that are not kept
    {
        const int c = tid & 63;
        if (c < cols)
            for (int e = ((S.nm2 + 1) >> 1) + (tid >> 6); e < ((S.nm2 + 1) >> 1) + K2 - S.nm2; e += BQ_NT / 64)
                X2[e * BQ_KS2 + c] = make_float2(0.f, 0.f);
    }
    __syncthreads();
    bq_fft_axis2<true>(X2, K2, tw2, tid);
    // a thread keeps its row; the even one of a pair packs Z(m), the odd one Z(K3 - m)
    {
        const int r = tid & (2 * BQ_NC - 1);
        const int j = r / K2, g2 = r - j * K2;
        const float2* x = X2 + g2 * BQ_KS2 + j * km;
        float2* z = buf + (r >> 1);
        const bool odd = (r & 1) != 0;
        constexpr int STEP = BQ_NT / (2 * BQ_NC), PM = (BQ_KAX / 2 + STEP) / STEP;
        const int mf = tid / (2 * BQ_NC);
        float2 zv[PM];
#pragma unroll
        for (int q = 0; q < PM; ++q) {
            const int m = mf + q * STEP;
            const float2 own = r < rows && m < km ? x[m] : make_float2(0.f, 0.f);
            const float2 oth = make_float2(__shfl_xor(own.x, 1, 64), __shfl_xor(own.y, 1, 64));
            zv[q] = odd ? make_float2(oth.x + own.y, own.x - oth.y) : make_float2(own.x - oth.y, own.y + oth.x);
        }
        __syncthreads();
        if (r < rows) {   // whole pairs: rows is even
#pragma unroll
            for (int q = 0; q < PM; ++q) {
                const int m = mf + q * STEP;
                if (odd ? m > 0 && 2 * m < K3 : 2 * m <= K3) z[(odd ? K3 - m : m) * BQ_KS] = zv[q];
            }
        }
    }
    __syncthreads();
    bq_fft_lines<true>(buf, K3, tw3, tid);
}

// Inverse transforms of a block's planes and, from LDS, the part of every
// atom's interpolation that lies on them: mpart[k1][i] for the plane h1 - k1
// (eq. matvec: the integral of the potential over the atom's distribution).
// With FIN also the three derivative sums, mpart[8 (1 + c) + k1][i].  Two
// lanes per (atom, plane), half of the axis-2 rows each, as in the spread.
template <bool FIN>
__global__ __launch_bounds__(BQ_NT) void k_bq_inv(BArgs a, const int2* __restrict__ units, int mode) {
    extern __shared__ float2 lds[];
    const int2 u = units[blockIdx.x];
    if (u.x < 0) return;
    const BStruct& S = a.st[u.x];
    BState& T = a.state[u.x];
    if (!bq_active(T, mode)) return;
    long long t0 = wall_clock64();
    __shared__ float2 tw3[BQ_KAX], tw2[BQ_KAX];
    __shared__ int first[BQ_PB], off[BQ_PB + 1];
    const int tid = threadIdx.x, n = S.n, p = a.p;
    const int K1 = S.K[0], K2 = S.K[1], K3 = S.K[2];
    const int g1a = u.y * S.pb, planes = min(S.pb, K1 - g1a);
    if (tid < K3) tw3[tid] = a.tw[S.tw_off[2] + tid];
    if (tid >= BQ_KAX && tid - BQ_KAX < K2) tw2[tid - BQ_KAX] = a.tw[S.tw_off[1] + tid - BQ_KAX];
    bq_ranges(slot_ptr<int>(a, S, S.slot.hstart), K1, n, p, g1a, planes, tid, first, off);
    bq_inverse_planes(a, S, g1a, planes, lds, tw2, tw3, tid);
    if (tid == 0) t0 = bq_lap(T, PH_FFT, t0);
    const float* bf = reinterpret_cast<const float*>(lds);
    const int* home = slot_ptr<int>(a, S, S.slot.home);
    const float* wts = slot_ptr<float>(a, S, S.slot.wts);
    const float* dwts = slot_ptr<float>(a, S, S.slot.dwts);
    float* mpart = slot_ptr<float>(a, S, S.slot.mpart);
    const int items = off[planes], hp = p >> 1, k20 = (tid & 1) * hp;
    const int rounds = (items + BQ_NT / 2 - 1) / (BQ_NT / 2);
    for (int rd = 0; rd < rounds; ++rd) {
        const int t = rd * (BQ_NT / 2) + (tid >> 1);
        const bool live = t < items;
        float s = 0.f, s2 = 0.f, s3 = 0.f, w1 = 0.f, dw1 = 0.f;
        int i = 0, k1 = 0;
        if (live) {
            int j = 0;
            while (t >= off[j + 1]) ++j;
            i = first[j] + (t - off[j]);
            if (i >= n) i -= n;
            const int4 hm = *reinterpret_cast<const int4*>(home + 4 * i);
            k1 = hm.x - (g1a + j);
            if (k1 < 0) k1 += K1;
            const float* w = wts + (size_t)i * 3 * QEQ_MAXP;
            const float* dw = dwts + (size_t)i * 3 * QEQ_MAXP;
            w1 = w[k1];
            if (FIN) dw1 = dw[k1];
            const float4 wa = *reinterpret_cast<const float4*>(w + 2 * QEQ_MAXP);
            const float4 wb = *reinterpret_cast<const float4*>(w + 2 * QEQ_MAXP + 4);
            const float w3[8] = {wa.x, wa.y, wa.z, wa.w, wb.x, wb.y, wb.z, wb.w};
            int g2 = hm.y - k20;
            if (g2 < 0) g2 += K2;
            const float* col[QEQ_MAXP];
#pragma unroll
            for (int k3 = 0; k3 < QEQ_MAXP; ++k3) {
                int g3 = hm.z - k3;
                if (g3 < 0) g3 += K3;
                col[k3] = bf + 2 * g3 * BQ_KS;
            }
            const int r0 = j * K2;
            for (int q = 0; q < hp; ++q) {
                const int at = r0 + g2;   // rows r and r ^ 1 share a complex value (r0 is even)
                float x = 0.f, x3 = 0.f;
#pragma unroll
                for (int k3 = 0; k3 < QEQ_MAXP; ++k3) {
                    if (k3 >= p) break;
                    const float g = col[k3][at];
                    x += w3[k3] * g;
                    if (FIN) x3 += dw[2 * QEQ_MAXP + k3] * g;
                }
                const float w2 = w[QEQ_MAXP + k20 + q];
                s += w2 * x;
                if (FIN) {
                    s2 += dw[QEQ_MAXP + k20 + q] * x;
                    s3 += w2 * x3;
                }
                g2 = g2 == 0 ? K2 - 1 : g2 - 1;
            }
        }
        s += __shfl_xor(s, 1, 64);
        if (FIN) {
            s2 += __shfl_xor(s2, 1, 64);
            s3 += __shfl_xor(s3, 1, 64);
        }
        if (live && (tid & 1) == 0) {
            mpart[(size_t)k1 * n + i] = w1 * s;
            if (FIN) {
                mpart[(size_t)(QEQ_MAXP + k1) * n + i] = dw1 * s;
                mpart[(size_t)(2 * QEQ_MAXP + k1) * n + i] = w1 * s2;
                mpart[(size_t)(3 * QEQ_MAXP + k1) * n + i] = w1 * s3;
            }
        }
    }
    if (tid == 0) bq_lap(T, PH_INTERP, t0);
}

// One plane d1 = -(p-1) .. p-1 of the mesh kernel Theta around the origin, for
// the self-correction.
__global__ __launch_bounds__(BQ_NT) void k_bq_theta(BArgs a, const int2* __restrict__ units) {
    extern __shared__ float2 lds[];
    const int2 u = units[blockIdx.x];
    const BStruct& S = a.st[u.x];
    BState& T = a.state[u.x];
    if (T.finished) return;
    const long long t0 = wall_clock64();
    __shared__ float2 tw3[BQ_KAX], tw2[BQ_KAX];
    const int tid = threadIdx.x, p = a.p, np = 2 * p - 1;
    const int K1 = S.K[0], K2 = S.K[1], K3 = S.K[2];
    const int d1 = u.y - (p - 1);
    if (tid < K3) tw3[tid] = a.tw[S.tw_off[2] + tid];
    if (tid >= BQ_KAX && tid - BQ_KAX < K2) tw2[tid - BQ_KAX] = a.tw[S.tw_off[1] + tid - BQ_KAX];
    __syncthreads();
    bq_inverse_planes(a, S, d1 < 0 ? d1 + K1 : d1, 1, lds, tw2, tw3, tid);
    const float* bf = reinterpret_cast<const float*>(lds);
    double* tab = slot_ptr<double>(a, S, S.slot.tab) + (size_t)u.y * np * np;
    for (int t = tid; t < np * np; t += BQ_NT) {
        const int d3 = t % np - (p - 1), d2 = t / np - (p - 1);
        const int g2 = d2 < 0 ? d2 + K2 : d2, g3 = d3 < 0 ? d3 + K3 : d3;
        tab[t] = (double)bf[2 * (g3 * BQ_KS + (g2 >> 1)) + (g2 & 1)];
    }
    if (tid == 0) bq_lap(T, PH_MESHPREP, t0);
}

// Mesh self-correction of 64 atoms, 16 lanes each.
template <int PC>
__global__ __launch_bounds__(256) void k_bq_self(BArgs a, const int2* __restrict__ units) {
    const int2 u = units[blockIdx.x];
    const BStruct& S = a.st[u.x];
    BState& T = a.state[u.x];
    if (T.finished) return;
    const long long t0 = wall_clock64();
    constexpr int NPM = SelfRows<PC>::NPM;
    __shared__ double tab[NPM * NPM * NPM];
    __shared__ SelfRows<PC> rows[16];
    const int np = 2 * a.p - 1;
    const double* tab_g = slot_ptr<double>(a, S, S.slot.tab);
    const double* frac = slot_ptr<double>(a, S, S.slot.frac);
    for (int t = threadIdx.x; t < np * np * np; t += 256) tab[t] = tab_g[t];
    SelfRows<PC>& w = rows[threadIdx.x >> 4];
    const int end = min(S.n, (u.y + 1) * 64);
    for (int i0 = u.y * 64; i0 < end; i0 += 16) {
        const int i = i0 + (threadIdx.x >> 4), ic = min(i, S.n - 1);
        if (i0 > u.y * 64) __syncthreads();   // the rows' LDS is free
        mesh_self_prepare<PC>(frac[3 * ic] * S.K[0], frac[3 * ic + 1] * S.K[1], frac[3 * ic + 2] * S.K[2], a.p, w);
        double v, g[3];
        mesh_self_sum<PC, true>(a.p, tab, w, &v, g);
        if (i < S.n && (threadIdx.x & 15) == 0) {
            slot_vec(a, S, V_DSELF)[i] += T.c_eta - v;
            double* sg = slot_ptr<double>(a, S, S.slot.selfgrad);
            for (int c = 0; c < 3; ++c) sg[3 * i + c] = g[c];
        }
    }
    if (threadIdx.x == 0) bq_lap(T, PH_MESHPREP, t0);
}

// ------------------------------------------------------------------ CG step
// One block per structure, one thread per atom: the atom's interpolation
// partials and pair sum, the sums of the product, and the CG step that follows
// it: residual and first direction
// (BQ_INIT), update and next direction (BQ_ITER), energies, mu, true residual,
// forces and the restart decision (BQ_FINAL).
template <int MODE>
__global__ __launch_bounds__(1024) void k_bq_step(BArgs a, const int* __restrict__ order) {
    constexpr bool FIN = MODE == BQ_FINAL;
    const int s = order[blockIdx.x];
    const BStruct& S = a.st[s];
    BState& T = a.state[s];
    if (!bq_active(T, MODE)) return;
    const long long t0 = wall_clock64();
    const int tid = threadIdx.x, n = S.n, p = a.p;
    const double Q = S.q_tot;
    if (MODE == BQ_INIT && (long long)T.nnz > S.pcap) {   // uniform
        if (tid == 0) {
            T.status = BQ_OVERFLOW;
            T.finished = 1;
            atomicSub(&a.count->running, 1);
        }
        return;
    }
    const bool live = tid < n;
    double* qv = slot_vec(a, S, V_Q);
    double* rv = slot_vec(a, S, V_R);
    double* pv = slot_vec(a, S, V_P);
    const double* src = MODE == BQ_ITER ? pv : qv;
    const float* mpart = slot_ptr<float>(a, S, S.slot.mpart);
    double vi = 0.0, yi = 0.0, Ji = 0.0, dsi = 0.0, chi = 0.0, dinv = 0.0, ri = 0.0, qi = 0.0;
    if (live) {
        float mp[QEQ_MAXP];
#pragma unroll
        for (int k = 0; k < QEQ_MAXP; ++k) mp[k] = k < p ? mpart[(size_t)k * n + tid] : 0.f;
        vi = src[tid];
        yi = slot_vec(a, S, V_Y)[tid];
        Ji = slot_vec(a, S, V_J)[tid];
        dsi = slot_vec(a, S, V_DSELF)[tid];
        dinv = slot_vec(a, S, V_DINV)[tid];
        if (MODE != BQ_ITER) chi = slot_vec(a, S, V_CHI)[tid];
        if (MODE == BQ_ITER) {
            ri = rv[tid];
            qi = qv[tid];
        }
#pragma unroll
        for (int k = 0; k < QEQ_MAXP; ++k) yi += (double)mp[k];
        if (FIN && a.forces) {
            double du[3] = {0.0, 0.0, 0.0};
            for (int c = 0; c < 3; ++c)
                for (int k = 0; k < p; ++k) du[c] += (double)mpart[(size_t)((c + 1) * QEQ_MAXP + k) * n + tid];
            if (a.self_corr) {
                const double* sg = slot_ptr<double>(a, S, S.slot.selfgrad);
                for (int c = 0; c < 3; ++c) du[c] -= 0.5 * vi * sg[3 * tid + c];
            }
            const double* fp = slot_ptr<double>(a, S, S.slot.fpair);
            double* f = a.forces + 3 * (size_t)(S.off + slot_ptr<int>(a, S, S.slot.perm)[tid]);
            for (int c = 0; c < 3; ++c) {
                double g = 0.0;
                for (int b = 0; b < 3; ++b) g += (double)S.K[b] * S.Hinv[c * 3 + b] * du[b];
                f[c] = -vi * g - vi * fp[3 * tid + c];
            }
        }
    }
    const double chi_norm = T.chi_norm;
    if (FIN) {
        double t5[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, g = 0.0;
        if (live) {
            const double y = yi + dsi * vi;
            const double sg = slot_vec(a, S, V_SIG)[tid];
            g = y + Ji * vi + chi;
            t5[0] = vi * y;
            t5[1] = slot_vec(a, S, V_CHIRAW)[tid] * vi;
            t5[2] = Ji * vi * vi;
            t5[3] = sg * sg * vi;
            t5[4] = g;
        }
        wg_sum<5>(t5);
        const double gmean = t5[4] / (double)n;
        double dv[1] = {live ? (g - gmean) * (g - gmean) : 0.0};
        wg_sum<1>(dv);
        const double tres = chi_norm > 0.0 ? sqrt(dv[0]) / chi_norm : sqrt(dv[0]);
        const double e_bg = -0.5 * S.bg_pref * (a.eta * a.eta * Q * Q - 2.0 * Q * t5[3]);
        const double e_elec = 0.5 * t5[0] + e_bg;
        const double e_qeq = e_elec + t5[1] + 0.5 * t5[2];
        const double mu = gmean - S.bg_pref * (a.eta * a.eta * Q - t5[3]);
        const bool gap = !(tres <= a.restart_thr);
        const bool conv = T.conv != 0;
        const bool stop = !conv || !gap || T.restarts >= 4 || T.iters >= a.max_iter;
        __syncthreads();   // every thread has read the state that thread 0 changes
        if (stop) {
            if (live) a.q_out[S.off + slot_ptr<int>(a, S, S.slot.perm)[tid]] = vi;
            if (tid == 0) {
                T.status = conv && !gap && isfinite(e_qeq) ? QEQ_OK : QEQ_NOT_CONVERGED;
                T.tres = tres;
                T.mu = mu;
                T.e_qeq = e_qeq;
                T.e_elec = e_elec;
                T.finished = 1;
                if (a.energies) {
                    a.energies[2 * (size_t)s] = e_qeq;
                    a.energies[2 * (size_t)s + 1] = e_elec;
                }
            }
        } else if (tid == 0) {
            T.restarts += 1;
            T.need_init = 1;
            T.cgdone = 0;
            atomicAdd(&a.count->restarts, 1);
            atomicAdd(&a.count->running, 1);
        }
    } else {
        double t2[2] = {0.0, 0.0}, y = 0.0;
        if (live) {
            y = yi + dsi * vi + Ji * vi;
            t2[0] = vi * y;
            t2[1] = y;
        }
        wg_sum<2>(t2);
        if (MODE == BQ_INIT) {
            const double shift = (T.chi_sum + t2[1]) / (double)n;
            double t4[4] = {0.0, 0.0, 0.0, 0.0};
            if (live) {
                ri = -chi - y + shift;
                rv[tid] = ri;
                t4[0] = dinv * ri;
                t4[1] = dinv * ri * ri;
                t4[2] = ri * ri;
                t4[3] = chi * vi;
            }
            wg_sum<4>(t4);
            const double c = t4[0] / T.dinv_sum;
            const double res = chi_norm > 0.0 ? sqrt(t4[2]) / chi_norm : sqrt(t4[2]);
            const bool first = a.q0 != nullptr && T.restarts == 0 && T.q0_rejected == 0 && T.iters == 0;
            const double e_start = 0.5 * t2[0] + t4[3];
            // a supplied start that is worse than the cold one is replaced by it
            const bool worse = first && (Q == 0.0 ? !(e_start < 0.0) : !(res <= 1.0));
            const bool done = res <= a.tol || !(res == res);
            const int it = T.iters;
            __syncthreads();
            if (live) {
                if (worse)
                    qv[tid] = Q / (double)n;
                else
                    pv[tid] = dinv * (ri - c);
            }
            if (tid == 0) {
                if (worse) {
                    T.q0_rejected = 1;
                } else {
                    T.need_init = 0;
                    T.rz = t4[1] - c * t4[0];
                    T.res = res;
                    T.conv = done;
                    if (done || it >= a.max_iter) {
                        T.cgdone = 1;
                        atomicSub(&a.count->running, 1);
                    }
                }
            }
        } else {
            const double rz = T.rz;
            const double alpha = rz / t2[0];
            const double ymean = t2[1] / (double)n;
            double t3[3] = {0.0, 0.0, 0.0};
            if (live) {
                qv[tid] = qi + alpha * vi;
                ri -= alpha * (y - ymean);
                rv[tid] = ri;
                t3[0] = dinv * ri;
                t3[1] = dinv * ri * ri;
                t3[2] = ri * ri;
            }
            wg_sum<3>(t3);
            const double c = t3[0] / T.dinv_sum;
            const double rz_new = t3[1] - c * t3[0];
            const double beta = rz_new / rz;
            const double res = chi_norm > 0.0 ? sqrt(t3[2]) / chi_norm : sqrt(t3[2]);
            const bool done = res <= a.tol || !(res == res);
            const int it = T.iters + 1;
            __syncthreads();
            if (live) pv[tid] = dinv * (ri - c) + beta * vi;
            if (tid == 0) {
                T.iters = it;
                T.rz = rz_new;
                T.res = res;
                T.conv = done;
                if (done || it >= a.max_iter) {
                    T.cgdone = 1;
                    atomicSub(&a.count->running, 1);
                }
            }
        }
    }
    if (tid == 0) bq_lap(T, PH_VEC, t0);
}

__global__ void k_bq_count_clear(BCount* c) { c->restarts = 0; }

// ------------------------------------------------------------------ host side
constexpr double PI_H = 3.14159265358979323846;

bool smooth_235_h(int n) {
    for (int f : {2, 3, 5})
        while (n % f == 0) n /= f;
    return n == 1;
}

bool length_compiled(int K) {
    switch (K) {
#define X(KK) case KK: return true;
        BQ_FOR_EACH_LEN(X)
#undef X
    }
    return false;
}

// |b(m)|^2 of the order-p cardinal B-spline (Essmann et al.), host FP64.
void bmod_h(int K, int p, float* out) {
    double c[QEQ_MAXP + 1] = {0};
    c[1] = 1.0;
    for (int nn = 3; nn <= p; ++nn) {
        const double inv = 1.0 / (nn - 1);
        for (int k = nn - 1; k >= 1; --k) c[k] = (k * c[k] + (nn - k) * c[k - 1]) * inv;
        c[0] = 0.0;
    }
    for (int m = 0; m < K; ++m) {
        double re = 0.0, im = 0.0;
        for (int k = 0; k <= p - 2; ++k) {
            const double ang = 2.0 * PI_H * (double)m * k / K;
            re += c[k + 1] * cos(ang);
            im += c[k + 1] * sin(ang);
        }
        const double d = re * re + im * im;
        out[m] = d > 1e-30 ? (float)(1.0 / d) : 0.f;
    }
}

void inv3_h(const double* H, double* Hi, double* det) {
    const double a = H[0], b = H[1], c = H[2], d = H[3], e = H[4], f = H[5], g = H[6], h = H[7], i = H[8];
    const double A = e * i - f * h, B = -(d * i - f * g), C = d * h - e * g;
    const double D = -(b * i - c * h), E = a * i - c * g, F = -(a * h - b * g);
    const double G = b * f - c * e, Hh = -(a * f - c * d), I = a * e - b * d;
    *det = a * A + b * B + c * C;
    const double r = 1.0 / *det;
    Hi[0] = A * r; Hi[1] = D * r; Hi[2] = G * r;
    Hi[3] = B * r; Hi[4] = E * r; Hi[5] = Hh * r;
    Hi[6] = C * r; Hi[7] = F * r; Hi[8] = I * r;
}

template <typename T>
int grow(T** p, size_t* cap, size_t count) {
    if (count <= *cap && *p) return QEQ_OK;
    if (*p) (void)hipFree(*p);
    *p = nullptr;
    *cap = 0;
    if (hipMalloc((void**)p, std::max<size_t>(count, 1) * sizeof(T)) != hipSuccess) return QEQ_ENOMEM;
    if (poisonable<T>) debug_poison(*p, count * sizeof(T));
    *cap = count;
    return QEQ_OK;
}

// Scratch of the structures that are solved together (1,024 structures of
// 32 .. 512 atoms: 1.6 GB).
constexpr size_t BQ_SCRATCH = (size_t)8 << 30;

}  // namespace qeqb

using namespace qeqb;

// Workspace of the batched path, owned by the plan.
struct BatchState {
    char* scratch = nullptr;
    size_t scratch_cap = 0;
    char* tables = nullptr;      // structures, states, units and transform tables of one wave of structures
    size_t tables_cap = 0;
    char* staging = nullptr;     // the same in pinned host memory: one copy a wave
    size_t staging_cap = 0;
    BCount* count_host = nullptr;   // pinned: counters of the chunks in flight
    hipEvent_t ev[2] = {nullptr, nullptr};
    hipEvent_t span[2] = {nullptr, nullptr};   // before a wave's first and after its last kernel
    double last_ms = 0.0;
    std::vector<BState> last_state;   // per-structure records of the last call
};

void batch_free(qeq_plan* pl) {
    BatchState* b = pl->batch;
    if (!b) return;
    if (b->scratch) (void)hipFree(b->scratch);
    if (b->tables) (void)hipFree(b->tables);
    if (b->staging) (void)hipHostFree(b->staging);
    if (b->count_host) (void)hipHostFree(b->count_host);
    for (hipEvent_t e : {b->ev[0], b->ev[1], b->span[0], b->span[1]})
        if (e) (void)hipEventDestroy(e);
    delete b;
    pl->batch = nullptr;
}

namespace {

BatchState* batch_state(qeq_plan* pl) {
    if (!pl->batch) pl->batch = new (std::nothrow) BatchState();
    return pl->batch;
}

// Units of work of one kernel: (structure, piece).  Blocks are dispatched to
// the 8 XCDs round-robin, so the units are dealt out such that every piece of a
// structure has the same block number modulo 8 in every kernel and finds what
// the previous kernel of the product wrote in its XCD's L2; short lists are
// filled up with (-1, 0).
void deal_units(const std::vector<int>& work, const std::vector<int>& pieces, int atoms, const std::vector<int>& xcd,
                std::vector<int2>& out, const std::vector<BStruct>* st = nullptr) {
    std::vector<int2> lane[8];
    for (size_t w = 0; w < work.size(); ++w) {
        // chunks of `atoms` atoms first, as pieces -1, -2, ...
        if (atoms)
            for (int c = 0; c * atoms < (*st)[work[w]].n; ++c) lane[xcd[w]].push_back(make_int2(work[w], -1 - c));
        for (int t = 0; t < pieces[w]; ++t) lane[xcd[w]].push_back(make_int2(work[w], t));
    }
    size_t most = 0;
    for (const auto& v : lane) most = std::max(most, v.size());
    out.assign(8 * most, make_int2(-1, 0));
    for (int x = 0; x < 8; ++x)
        for (size_t t = 0; t < lane[x].size(); ++t) out[8 * t + x] = lane[x][t];
}

// One wave: the structures `work` (indices into st), whose slots start at
// their st.base; the device states come back in `state`.
int run_wave(qeq_plan* pl, BatchState* b, BArgs& a, std::vector<BStruct>& st, const std::vector<int>& work,
             const std::vector<float2>& twh, const std::vector<float>& bmh, std::vector<BState>& state) {
    hipStream_t stream = pl->stream;
    const int ns = (int)work.size();
    std::vector<int> nA(ns), nB(ns), nC(ns), nP(ns), nG(ns), nS(ns), nT(ns), xcd(ns);
    double load[8] = {0.0};
    for (int w = 0; w < ns; ++w) {
        const BStruct& S = st[work[w]];
        nA[w] = (S.K[0] + S.pf - 1) / S.pf;
        nC[w] = (S.K[0] + S.pb - 1) / S.pb;
        nB[w] = (S.nm2 * S.km + BQ_NC - 1) / BQ_NC;
        nP[w] = (S.n + BQ_PAIR_ATOMS - 1) / BQ_PAIR_ATOMS;
        nG[w] = (S.nhalf + BQ_GREEN - 1) / BQ_GREEN;
        nS[w] = (S.n + 63) / 64;
        nT[w] = 2 * a.p - 1;
        xcd[w] = (int)(std::min_element(load, load + 8) - load);   // longest first: balanced
        load[xcd[w]] += S.nhalf;
    }
    std::vector<int2> uA, uB, uC, uV, uP, uG, uS, uT;
    deal_units(work, nA, 0, xcd, uA);
    deal_units(work, nB, 0, xcd, uB);
    deal_units(work, nC, 0, xcd, uC);
    deal_units(work, nB, BQ_NT / BQ_L, xcd, uV, &st);   // with the pair products
    auto plain = [&](const std::vector<int>& pieces, std::vector<int2>& out) {
        for (int w = 0; w < ns; ++w)
            for (int t = 0; t < pieces[w]; ++t) out.push_back(make_int2(work[w], t));
    };
    plain(nP, uP);
    plain(nG, uG);
    if (a.self_corr) {
        plain(nS, uS);
        plain(nT, uT);
    }
    // tables: one staging buffer, one copy
    const int n_struct = (int)st.size();
    size_t o = 0;
    auto place = [&](size_t bytes) {
        const size_t at = o;
        o = align256(o + bytes);
        return at;
    };
    const size_t oSt = place(sizeof(BStruct) * n_struct), oState = place(sizeof(BState) * n_struct),
                 oCount = place(sizeof(BCount)), oOrder = place(sizeof(int) * ns), oTw = place(sizeof(float2) * twh.size()),
                 oBm = place(sizeof(float) * bmh.size()), oA = place(sizeof(int2) * uA.size()),
                 oB = place(sizeof(int2) * uB.size()), oV = place(sizeof(int2) * uV.size()),
                 oC = place(sizeof(int2) * uC.size()), oP = place(sizeof(int2) * uP.size()),
                 oG = place(sizeof(int2) * uG.size()), oS = place(sizeof(int2) * uS.size()),
                 oT = place(sizeof(int2) * uT.size());
    if (o > b->staging_cap) {
        if (b->staging) (void)hipHostFree(b->staging);
        b->staging = nullptr;
        b->staging_cap = 0;
        if (hipHostMalloc((void**)&b->staging, o + o / 4) != hipSuccess) {
            b->staging = nullptr;
            return QEQ_ENOMEM;
        }
        b->staging_cap = o + o / 4;
    }
    QEQ_TRY(grow(&b->tables, &b->tables_cap, o));
    if (!b->count_host && hipHostMalloc((void**)&b->count_host, 2 * sizeof(BCount)) != hipSuccess) {
        b->count_host = nullptr;
        return QEQ_ENOMEM;
    }
    for (hipEvent_t& e : b->ev)
        if (!e) QEQ_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    for (hipEvent_t& e : b->span)
        if (!e) QEQ_HIP(hipEventCreate(&e));
    memset(b->staging + oState, 0, sizeof(BState) * n_struct);
    const BCount c0 = {ns, 0};
    auto put = [&](size_t at, const void* from, size_t bytes) {
        if (bytes) memcpy(b->staging + at, from, bytes);
    };
    put(oSt, st.data(), sizeof(BStruct) * n_struct);
    put(oCount, &c0, sizeof(c0));
    put(oOrder, work.data(), sizeof(int) * ns);
    put(oTw, twh.data(), sizeof(float2) * twh.size());
    put(oBm, bmh.data(), sizeof(float) * bmh.size());
    put(oA, uA.data(), sizeof(int2) * uA.size());
    put(oB, uB.data(), sizeof(int2) * uB.size());
    put(oV, uV.data(), sizeof(int2) * uV.size());
    put(oC, uC.data(), sizeof(int2) * uC.size());
    put(oP, uP.data(), sizeof(int2) * uP.size());
    put(oG, uG.data(), sizeof(int2) * uG.size());
    put(oS, uS.data(), sizeof(int2) * uS.size());
    put(oT, uT.data(), sizeof(int2) * uT.size());
    QEQ_HIP(hipMemcpyAsync(b->tables, b->staging, o, hipMemcpyHostToDevice, stream));
    a.st = (const BStruct*)(b->tables + oSt);
    a.state = (BState*)(b->tables + oState);
    a.count = (BCount*)(b->tables + oCount);
    a.tw = (const float2*)(b->tables + oTw);
    a.bmod = (const float*)(b->tables + oBm);
    a.scratch = b->scratch;
    const int* order = (const int*)(b->tables + oOrder);
    const int2 *dA = (const int2*)(b->tables + oA), *dB = (const int2*)(b->tables + oB),
               *dV = (const int2*)(b->tables + oV), *dC = (const int2*)(b->tables + oC),
               *dP = (const int2*)(b->tables + oP), *dG = (const int2*)(b->tables + oG),
               *dS = (const int2*)(b->tables + oS), *dT = (const int2*)(b->tables + oT);
    size_t shA = 0, shB = 0, shC = 0;
    for (int s : work) {
        const BStruct& S = st[s];
        shC = std::max(shC, bq_lds_inv(S.K[1], S.K[2]));
        shA = std::max(shA, bq_lds_fwd(S.K[1], S.K[2], S.pf));
        shB = std::max(shB, bq_lds_lines(S.K[0]));
    }
    auto window = [](const void* fn, size_t sh) {
        return sh <= 65536 ? QEQ_OK
                           : qeq_check(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh));
    };
    QEQ_TRY(window((const void*)k_bq_fwd, shA));
    QEQ_TRY(window((const void*)k_bq_inv<false>, shC));
    QEQ_TRY(window((const void*)k_bq_inv<true>, shC));
    QEQ_TRY(window((const void*)k_bq_theta, shC));
    // --- set-up
    QEQ_HIP(hipEventRecord(b->span[0], stream));
    hipLaunchKernelGGL(k_bq_stage, dim3(ns), dim3(1024), 0, stream, a, order);
    hipLaunchKernelGGL(k_bq_pairs, dim3((unsigned)uP.size()), dim3(256), 0, stream, a, dP);
    hipLaunchKernelGGL(k_bq_green, dim3((unsigned)uG.size()), dim3(256), 0, stream, a, dG);
    if (a.self_corr) {
        hipLaunchKernelGGL(k_bq_cols<true>, dim3((unsigned)uB.size()), dim3(BQ_NT), shB, stream, a, dB, (int)BQ_FINAL);
        hipLaunchKernelGGL(k_bq_theta, dim3((unsigned)uT.size()), dim3(BQ_NT), shC, stream, a, dT);
        if (a.p == 6)
            hipLaunchKernelGGL(k_bq_self<6>, dim3((unsigned)uS.size()), dim3(256), 0, stream, a, dS);
        else
            hipLaunchKernelGGL(k_bq_self<0>, dim3((unsigned)uS.size()), dim3(256), 0, stream, a, dS);
    }
    QEQ_TRY(qeq_check(hipGetLastError()));
    auto product = [&](int mode) {
        hipLaunchKernelGGL(k_bq_fwd, dim3((unsigned)uA.size()), dim3(BQ_NT), shA, stream, a, dA, mode);
        hipLaunchKernelGGL(k_bq_cols<false>, dim3((unsigned)uV.size()), dim3(BQ_NT), shB, stream, a, dV, mode);
        if (mode == BQ_FINAL) {
            hipLaunchKernelGGL(k_bq_inv<true>, dim3((unsigned)uC.size()), dim3(BQ_NT), shC, stream, a, dC, mode);
            hipLaunchKernelGGL(k_bq_step<BQ_FINAL>, dim3(ns), dim3(1024), 0, stream, a, order);
        } else {
            hipLaunchKernelGGL(k_bq_inv<false>, dim3((unsigned)uC.size()), dim3(BQ_NT), shC, stream, a, dC, mode);
            if (mode == BQ_INIT)
                hipLaunchKernelGGL(k_bq_step<BQ_INIT>, dim3(ns), dim3(1024), 0, stream, a, order);
            else
                hipLaunchKernelGGL(k_bq_step<BQ_ITER>, dim3(ns), dim3(1024), 0, stream, a, order);
        }
        return qeq_check(hipGetLastError());
    };
    auto counters = [&](int slot) -> int {
        QEQ_HIP(hipMemcpyAsync(&b->count_host[slot], a.count, sizeof(BCount), hipMemcpyDeviceToHost, stream));
        QEQ_HIP(hipEventRecord(b->ev[slot], stream));
        return QEQ_OK;
    };
    for (int round = 0;; ++round) {
        QEQ_TRY(product(BQ_INIT));
        if (round == 0 && a.q0) QEQ_TRY(product(BQ_INIT));   // rejected starting charges
        // Chunks of iterations; the counter of each chunk is read while the
        // next one runs, so the stream never waits for the host and at most
        // one chunk of early-returning blocks is launched in vain.
        constexpr int CHUNK = 3;
        int slot = 0;
        bool first = true;
        for (int it = 0; it < a.max_iter; it += CHUNK) {
            for (int t = 0; t < CHUNK; ++t) QEQ_TRY(product(BQ_ITER));
            QEQ_TRY(counters(slot));
            if (!first) {
                QEQ_HIP(hipEventSynchronize(b->ev[slot ^ 1]));
                if (b->count_host[slot ^ 1].running == 0) break;
            }
            first = false;
            slot ^= 1;
        }
        QEQ_TRY(product(BQ_FINAL));
        QEQ_TRY(counters(0));
        QEQ_HIP(hipEventSynchronize(b->ev[0]));
        if (b->count_host[0].restarts == 0) break;
        hipLaunchKernelGGL(k_bq_count_clear, dim3(1), dim3(1), 0, stream, a.count);
        QEQ_TRY(qeq_check(hipGetLastError()));
    }
    QEQ_HIP(hipEventRecord(b->span[1], stream));
    QEQ_HIP(hipMemcpyAsync(b->staging + oState, a.state, sizeof(BState) * n_struct, hipMemcpyDeviceToHost, stream));
    QEQ_HIP(hipStreamSynchronize(stream));
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, b->span[0], b->span[1]) == hipSuccess) b->last_ms += ms;
    const BState* back = (const BState*)(b->staging + oState);
    for (int s : work) state[s] = back[s];
    return QEQ_OK;
}

int batched_impl(qeq_plan* pl, int n_struct, const int32_t* offs, const double* pos, const double* cells,
                 const double* sigma, const double* J, const double* chi, const double* q_tot, const double* q0,
                 double* q, double* energies, double* forces, qeq_stats* stats) {
    if (n_struct < 1 || !offs || !pos || !cells || !sigma || !J || !chi || !q_tot || !q) return QEQ_EINVAL;
    for (int s = 0; s < n_struct; ++s)
        if (offs[s] < 0 || offs[s + 1] < offs[s]) return QEQ_EINVAL;
    BatchState* b = batch_state(pl);
    if (!b) return QEQ_ENOMEM;
    const qeq_params& prm = pl->prm;
    const int p = prm.spline_order;
    const double rc = prm.r_cut;
    std::vector<BStruct> st(n_struct);
    std::vector<int> hstatus(n_struct, QEQ_OK);
    std::vector<int> Ks;                    // distinct axis lengths
    std::vector<double> cost(n_struct, 0.0);
    for (int s = 0; s < n_struct; ++s) {
        BStruct& S = st[s];
        memset(&S, 0, sizeof(S));
        const int n = offs[s + 1] - offs[s];
        S.n = n;
        S.off = offs[s];
        const double* cell = cells + 9 * (size_t)s;
        bool ok = n >= 1 && isfinite(q_tot[s]);
        for (int t = 0; t < 9; ++t) ok = ok && isfinite(cell[t]);
        double det = 0.0;
        if (ok) {
            inv3_h(cell, S.Hinv, &det);
            ok = det > 0.0 && isfinite(det);
        }
        if (!ok) {
            hstatus[s] = QEQ_EINVAL;
            continue;
        }
        if (n > QEQ_BATCH_NMAX) {
            hstatus[s] = QEQ_EPLAN;
            continue;
        }
        for (int t = 0; t < 9; ++t) S.H[t] = cell[t];
        S.vol = det;
        double Mm[9];
        for (int x = 0; x < 3; ++x)
            for (int y = 0; y < 3; ++y) {
                double v = 0.0;
                for (int c = 0; c < 3; ++c) v += S.Hinv[c * 3 + x] * S.Hinv[c * 3 + y];
                Mm[x * 3 + y] = v;
            }
        S.M[0] = Mm[0]; S.M[1] = Mm[4]; S.M[2] = Mm[8];
        S.M[3] = Mm[1]; S.M[4] = Mm[2]; S.M[5] = Mm[5];
        double widths[3], lengths[3];
        int K[3];
        bool gok = true;
        for (int x = 0; x < 3; ++x) {
            widths[x] = 1.0 / sqrt(Mm[x * 3 + x]);
            lengths[x] = sqrt(cell[3 * x] * cell[3 * x] + cell[3 * x + 1] * cell[3 * x + 1] +
                              cell[3 * x + 2] * cell[3 * x + 2]);
            if (prm.grid[0] > 0) {
                K[x] = prm.grid[x];
            } else {
                int m = (int)ceil(lengths[x] / prm.max_spacing - 1e-12);
                m = std::max(m, 12);
                m = (m + 3) / 4 * 4;
                while (!smooth_235_h(m)) m += 4;
                K[x] = m;
            }
            gok = gok && K[x] >= 2 * p && K[x] >= 12 && K[x] <= BQ_KAX && K[x] % 4 == 0 && length_compiled(K[x]);
            S.K[x] = K[x];
            S.rho[x] = rc / widths[x];
            gok = gok && S.rho[x] <= 4.0;
        }
        if (!gok) {
            hstatus[s] = QEQ_EPLAN;
            continue;
        }
        const double kcut = sqrt(2.0 * 30.0 * 0.69314718055994530942) / prm.eta;
        S.km = std::min(K[2] / 2 + 1, (int)std::min(1e6, kcut * lengths[2] / (2 * PI_H)) + 1);
        S.nm2 = std::min(K[1], 2 * (int)std::min(1e6, kcut * lengths[1] / (2 * PI_H)) + 1);
        S.nhalf = K[0] * S.nm2 * S.km;
        S.green_pref = 4.0 * PI_H / det;
        S.bg_pref = 2.0 * PI_H / det;
        S.q_tot = q_tot[s];
        // second split for C_eta (same ranges as the single-structure host sum)
        S.zeta = std::max(prm.eta, 0.3 * cbrt(det));
        const double X = 6.5 * sqrt(2.0);
        const double kmx = X / S.zeta, rmx = X * S.zeta;
        for (int x = 0; x < 3; ++x) {
            S.mm[x] = (int)ceil(kmx * lengths[x] / (2 * PI_H)) + 1;
            S.nn[x] = (int)ceil(rmx / widths[x]) + 1;
        }
        for (int x = 0; x < 3; ++x)
            if (std::find(Ks.begin(), Ks.end(), K[x]) == Ks.end()) Ks.push_back(K[x]);
        S.pb = bq_planes_inv(K[0], K[1], S.km, p);
        S.pf = bq_planes_fwd(S.pb, K[1], K[2]);
        // pair capacity: mean neighbour count of a uniform density plus a
        // generous Poisson tail
        const double dens = n / det;
        const double mean = dens * 4.0 / 3.0 * PI_H * rc * rc * rc;
        const long long row = (long long)ceil(mean + 6.0 * sqrt(mean) + 16.0);
        S.pcap = (long long)n * std::min<long long>(row, (long long)n * 27);
        cost[s] = (double)K[0] * K[1] * K[2] * 12.0 + (double)n * (216.0 + mean);
    }
    // tables for the distinct axis lengths
    std::vector<float2> twh;
    std::vector<float> bmh;
    std::vector<int> tw_off(Ks.size()), bm_off(Ks.size());
    for (size_t u = 0; u < Ks.size(); ++u) {
        const int K = Ks[u];
        tw_off[u] = (int)twh.size();
        bm_off[u] = (int)bmh.size();
        for (int j = 0; j < K; ++j) {
            const double ang = -2.0 * PI_H * (double)j / (double)K;
            twh.push_back(make_float2((float)cos(ang), (float)sin(ang)));
        }
        std::vector<float> bm(K);
        bmod_h(K, p, bm.data());
        bmh.insert(bmh.end(), bm.begin(), bm.end());
    }
    std::vector<int> work;
    for (int s = 0; s < n_struct; ++s) {
        if (hstatus[s] != QEQ_OK) continue;
        BStruct& S = st[s];
        for (int x = 0; x < 3; ++x) {
            const size_t u = std::find(Ks.begin(), Ks.end(), S.K[x]) - Ks.begin();
            S.tw_off[x] = tw_off[u];
            S.bm_off[x] = bm_off[u];
        }
        work.push_back(s);
    }
    // longest first
    std::stable_sort(work.begin(), work.end(), [&](int x, int y) { return cost[x] > cost[y]; });

    std::vector<BState> state(n_struct);
    memset(state.data(), 0, sizeof(BState) * n_struct);
    for (int s = 0; s < n_struct; ++s) state[s].status = hstatus[s];
    BArgs a;
    memset(&a, 0, sizeof(a));
    a.p = p;
    a.self_corr = prm.self_correction;
    a.max_iter = prm.max_iter;
    a.tol = prm.tol;
    a.eta = prm.eta;
    a.rc2 = rc * rc;
    a.restart_thr = 2.0 * std::max(prm.tol, 1e-7);
    a.pos = pos;
    a.sigma = sigma;
    a.J = J;
    a.chi = chi;
    a.q0 = q0;
    a.q_out = q;
    a.energies = energies;
    a.forces = forces;
    int rc2 = QEQ_OK;
    // structures whose pair list overflowed go again with the measured size
    for (int round = 0; round < 2 && !work.empty() && rc2 == QEQ_OK; ++round) {
        std::vector<int> again;
        // as many structures at a time as BQ_SCRATCH holds (at least one); half
        // of that after a failed allocation
        size_t limit = BQ_SCRATCH;
        for (size_t w0 = 0; w0 < work.size() && rc2 == QEQ_OK;) {
            size_t used = 0, w1 = w0;
            for (; w1 < work.size(); ++w1) {
                BStruct& S = st[work[w1]];
                const size_t bytes = slot_layout(S.slot, (size_t)S.n, (size_t)S.nhalf, (size_t)S.pcap);
                if (w1 > w0 && used + bytes > limit) break;
                S.base = used;
                used += bytes;
            }
            rc2 = grow(&b->scratch, &b->scratch_cap, used);
            if (rc2 == QEQ_ENOMEM && w1 - w0 > 1) {
                (void)hipGetLastError();
                limit = used / 2;
                rc2 = QEQ_OK;
                continue;
            }
            if (rc2 != QEQ_OK) break;
            const std::vector<int> wave(work.begin() + w0, work.begin() + w1);
            rc2 = run_wave(pl, b, a, st, wave, twh, bmh, state);
            for (int s : wave)
                if (rc2 == QEQ_OK && state[s].status == BQ_OVERFLOW) {
                    again.push_back(s);
                    st[s].pcap = (long long)state[s].nnz;
                }
            w0 = w1;
        }
        work.swap(again);
    }
    if (rc2 != QEQ_OK) {
        (void)hipStreamSynchronize(pl->stream);   // nothing of this call stays in flight
        return rc2;
    }
    b->last_state = state;
    int worst = QEQ_OK;
    for (int s = 0; s < n_struct; ++s) {
        int code = state[s].status;
        if (code == BQ_OVERFLOW) code = QEQ_ENOMEM;
        if (stats) {
            qeq_stats& o = stats[s];
            memset(&o, 0, sizeof(o));
            o.status = code;
            o.iters = state[s].iters;
            o.rel_resid = state[s].res;
            o.true_rel_resid = state[s].tres;
            o.mu = state[s].mu;
            o.e_qeq = state[s].e_qeq;
            o.e_elec = state[s].e_elec;
            o.q0_rejected = state[s].q0_rejected;
        }
        if (code < 0) {
            if (worst >= 0 || code < worst) worst = code;
        } else if (code > 0 && worst == QEQ_OK) {
            worst = code;
        }
    }
    return worst;
}

}  // namespace

extern "C" {

int qeq_solve_batched(qeq_plan* plan, int32_t n_struct, const int32_t* atom_offsets, const double* pos,
                      const double* cells, const double* sigma, const double* J, const double* chi,
                      const double* q_tot, const double* q0, double* q, double* energies, double* forces,
                      qeq_stats* stats) {
    if (!plan) return QEQ_EINVAL;
    plan->tape_valid = false;
    plan->np_valid = false;
    plan->geom_valid = false;
    plan->ew_active = false;
    plan->pw_active = false;
    np_leave(plan);
    return batched_impl(plan, n_struct, atom_offsets, pos, cells, sigma, J, chi, q_tot, q0, q, energies, forces,
                        stats);
}

int qeq_batched_config(qeq_plan* plan, int32_t threads, int32_t wg_per_cu) {
    if (!plan) return QEQ_EINVAL;
    // the launch shapes of an earlier kernel, one persistent workgroup per
    // structure; what it refused stays refused, and nothing depends on the rest
    if (threads != 1024) return QEQ_EINVAL;
    if (wg_per_cu < 1 || wg_per_cu > 8) return QEQ_EINVAL;
    return QEQ_OK;
}

int qeq_batched_phase_us(qeq_plan* plan, int32_t n_struct, double* us) {
    if (!plan || !plan->batch || !us || n_struct < 0) return QEQ_EINVAL;
    const std::vector<BState>& v = plan->batch->last_state;
    if ((size_t)n_struct > v.size()) return QEQ_EINVAL;
    for (int s = 0; s < n_struct; ++s) {
        double* row = us + (size_t)s * (PH_COUNT + 1);
        row[PH_COUNT] = 0.0;
        for (int k = 0; k < PH_COUNT; ++k) {
            row[k] = (double)v[s].ticks[k] * 0.01;
            row[PH_COUNT] += row[k];
        }
    }
    return PH_COUNT + 1;
}

double qeq_batched_last_ms(qeq_plan* plan, int32_t reset) {
    if (!plan || !plan->batch) return 0.0;
    const double v = plan->batch->last_ms;
    if (reset) plan->batch->last_ms = 0.0;
    return v;
}

}  // extern "C"
