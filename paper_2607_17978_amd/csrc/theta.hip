// Tables of the mesh kernel Theta(d) on the offsets |d_a| < p, and of its six
// strain derivatives, for the self-correction: the inverse transform of the
// Green's function at (2p - 1)^3 points only,
//   Theta(d) = sum_m G(m) exp(2 pi i m.d / K),
// axis by axis: per m3 plane axis 1 and then axis 2 onto the 2p - 1 offsets
// (k_theta_plane), then axis 3 (k_theta_tab).  G is real, so along axis 1 the
// cosine and sine sums serve both signs of d_1.  The sums are in FP64 (G in
// FP32, as in the products).
//
// A table took five launches with full-size transforms through memory (write G,
// axis 1, axis 2, axis 3, pick the offsets), the six strain tables thirty; now
// two each: 12 us and 17 us at 40 x 60 x 60 where they took 19 and 116, and two
// steps of a 500-atom triclinic cell with virials 2.83 -> 2.65 ms.  One table /
// six at order 6, us, with the transforms and now: 96^3 29 / 238 and 21 / 24,
// 192^3 58 / 368 and 29 / 93, 320^3 230 / 1,404 and 73 / 310, 384^3 1,935 / 11,600
// and 105 / 628, 512 x 512 x 12 665 / 3,966 and 50 / 57.  Bound by the FP64
// multiply-adds, 2 p a mode, and the Green's function.
#include <algorithm>

#include "mesh_passes.h"

namespace {

constexpr int TH_W = 8;                  // waves of a plane block
constexpr int TH_BLOCKS = 512;           // plane blocks that the launch aims at
constexpr int TH_NP = 2 * QEQ_MAXP - 1;  // most offsets along an axis

// Component order of symmetric 3x3 tensors: 00, 11, 22, 01, 02, 12.
__device__ __forceinline__ void sym_pair(int comp, int& a, int& b) {
    a = comp < 3 ? comp : (comp == 5 ? 1 : 0);
    b = comp < 3 ? comp : (comp == 3 ? 1 : 2);
}

// G(m) of the table (comp < 0), or G(m) d ln G / d eps_ab.
__device__ __forceinline__ float theta_green(const KParams& k, int m1, int m2, int m3, const float* b1,
                                             const float* b2, const float* b3, int comp) {
    const float g = green_value(k, m1, m2, m3, b1, b2, b3);
    if (comp < 0 || g == 0.f) return g;
    float kv[3];
    const float k2 = mode_kvec(k, m1, m2, m3, kv);
    const float eta = (float)k.eta;
    int a, b;
    sym_pair(comp, a, b);
    return g * ((a == b ? -1.f : 0.f) + 2.f * (1.f / k2 + 0.5f * eta * eta) * kv[a] * kv[b]);
}

// Block (m3, table, z): 64 columns m2 at a time, a lane each; the waves share
// m1 and add up through LDS; then a thread per (d_1, d_2) takes the columns in.
// Every gridDim.z-th group of 64 columns.
// T[table][m3][d_1][d_2].
__global__ __launch_bounds__(64 * TH_W) void k_theta_plane(KParams k, const float* __restrict__ b1,
                                                           const float* __restrict__ b2,
                                                           const float* __restrict__ b3, int comp0,
                                                           double2* __restrict__ T) {
    extern __shared__ double2 sm[];
    const int K1 = k.K1, K2 = k.K2, p = k.p, np = 2 * p - 1;
    double2* e1 = sm;                                          // exp(2 pi i j / K1)
    double2* e2 = e1 + K1;
    double* S = reinterpret_cast<double*>(e2 + K2);            // [wave][2p][64]
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int m3 = blockIdx.x, comp = comp0 + (int)blockIdx.y;
    for (int j = tid; j < K1 + K2; j += 64 * TH_W) {
        double sn, cs;
        sincospi(2.0 * (j < K1 ? (double)j / K1 : (double)(j - K1) / K2), &sn, &cs);
        e1[j] = make_double2(cs, sn);
    }
    __syncthreads();
    const int od1 = tid / np - (p - 1), od2 = tid - (tid / np) * np - (p - 1);   // offsets of this thread's output
    const bool out = tid < np * np;
    double2 acc = make_double2(0.0, 0.0);
    for (int c0 = 64 * blockIdx.z; c0 < K2; c0 += 64 * gridDim.z) {
        const int m2 = c0 + lane;
        const bool in = m2 < K2 && m2_kept(k, m2);
        double C[QEQ_MAXP], D[QEQ_MAXP];
#pragma unroll
        for (int d = 0; d < QEQ_MAXP; ++d) C[d] = D[d] = 0.0;
        for (int m1 = w; m1 < K1; m1 += TH_W) {
            const double g = in ? (double)theta_green(k, m1, m2, m3, b1, b2, b3, comp) : 0.0;
            int j = 0;   // m1 d mod K1
#pragma unroll
            for (int d = 0; d < QEQ_MAXP; ++d) {
                if (d < p) {
                    const double2 e = e1[j];
                    C[d] += g * e.x;
                    D[d] += g * e.y;
                    j += m1;
                    j = j >= K1 ? j - K1 : j;
                }
            }
        }
#pragma unroll
        for (int d = 0; d < QEQ_MAXP; ++d) {
            if (d < p) {
                S[((size_t)w * 2 * p + 2 * d) * 64 + lane] = C[d];
                S[((size_t)w * 2 * p + 2 * d + 1) * 64 + lane] = D[d];
            }
        }
        __syncthreads();
        for (int t = tid; t < 2 * p * 64; t += 64 * TH_W) {
            double s = 0.0;
            for (int v = 0; v < TH_W; ++v) s += S[(size_t)v * 2 * p * 64 + t];
            S[t] = s;   // the first wave's part, read by this thread only
        }
        __syncthreads();
        if (out) {
            const int ad = abs(od1), cols = min(64, K2 - c0);
            const double sg = od1 < 0 ? -1.0 : 1.0;
            const double *Cs = S + (size_t)2 * ad * 64, *Ds = Cs + 64;
            const int dm = od2 < 0 ? od2 + K2 : od2;   // d_2 mod K2
            int j = (int)((long long)c0 * dm % K2);    // m2 d_2 mod K2
            for (int x = 0; x < cols; ++x) {
                const double2 e = e2[j];
                const double re = Cs[x], im = sg * Ds[x];
                acc.x += re * e.x - im * e.y;
                acc.y += re * e.y + im * e.x;
                j += dm;
                j = j >= K2 ? j - K2 : j;
            }
        }
        __syncthreads();
    }
    if (out) T[(((size_t)blockIdx.y * k.K3h + m3) * gridDim.z + blockIdx.z) * np * np + tid] = acc;
}

// tab[table][d_1][d_2][d_3] = sum over m3 of the half spectrum; block (d_1 d_2,
// table), a thread per d_3 and part of the m3.
__global__ __launch_bounds__(256) void k_theta_tab(KParams k, int nz, const double2* __restrict__ T,
                                                   double* __restrict__ tab) {
    __shared__ double red[16][16];
    const int np = 2 * k.p - 1, x = blockIdx.x, l = threadIdx.x & 15, q = threadIdx.x >> 4;
    const int d3 = l - (k.p - 1);
    double s = 0.0;
    if (l < np)
        for (int m3 = q; m3 < k.K3h; m3 += 16) {
            const double2* pl = T + ((size_t)blockIdx.y * k.K3h + m3) * nz * np * np + x;
            double2 t = pl[0];
            for (int z = 1; z < nz; ++z) {
                t.x += pl[(size_t)z * np * np].x;
                t.y += pl[(size_t)z * np * np].y;
            }
            double sn, cs;
            sincospi(2.0 * (double)(m3 * d3) / k.K3, &sn, &cs);
            s += (m3 == 0 ? 1.0 : 2.0) * (t.x * cs - t.y * sn);
        }
    red[q][l] = s;
    __syncthreads();
    if (threadIdx.x >= np) return;
    double v = 0.0;
    for (int u = 0; u < 16; ++u) v += red[u][threadIdx.x];
    // to FP32, the precision of G and of the mesh products that the table corrects
    tab[((size_t)blockIdx.y * np * np + x) * np + threadIdx.x] = (double)(float)v;
}

}  // namespace

// The table of Theta (strain = false) or the six of its strain derivatives,
// one after the other.
int launch_theta(qeq_plan* pl, bool strain, double* tab) {
    const KParams& k = pl->kp;
    const int np = 2 * k.p - 1, nt = strain ? 6 : 1;
    // With few planes their columns go to blocks of their own: two blocks a CU
    // (one table, a block a plane: 192^3 60 us at order 6 and 67 at order 8, where
    // the transforms took 58 and 57; 512 x 512 x 12 319 us).
    const int groups = (k.K2 + 63) / 64, planes = k.K3h * nt;
    const int nz = std::max(1, std::min(groups, (TH_BLOCKS + planes - 1) / planes));
    const size_t need = (size_t)planes * nz * np * np * 2;
    if (need > pl->theta_cap) {
        pl->theta_cap = 0;
        if (pl->theta_plane) (void)hipFree(pl->theta_plane);
        pl->theta_plane = nullptr;
        if (hipMalloc((void**)&pl->theta_plane, sizeof(double) * need) != hipSuccess) return QEQ_ENOMEM;
        debug_poison(pl->theta_plane, sizeof(double) * need);
        pl->theta_cap = need;
    }
    double2* T = reinterpret_cast<double2*>(pl->theta_plane);
    const size_t sh = sizeof(double2) * (k.K1 + k.K2) + sizeof(double) * TH_W * 2 * k.p * 64;
    QEQ_HIP(hipFuncSetAttribute((const void*)k_theta_plane, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh));
    hipLaunchKernelGGL(k_theta_plane, dim3(k.K3h, nt, nz), dim3(64 * TH_W), sh, pl->stream, k, pl->bmod[0], pl->bmod[1],
                       pl->bmod[2], strain ? 0 : -1, T);
    hipLaunchKernelGGL(k_theta_tab, dim3(np * np, nt), dim3(256), 0, pl->stream, k, nz, T, tab);
    return qeq_check(hipGetLastError());
}
