// Reciprocal-space part of the matrix-vector product (paper, "Electrostatics
// Solvers", eq. matvec): B-spline charge spreading, 3-D real-to-complex FFT,
// multiplication by the Gaussian-screened Green's function, inverse FFT.
//
// Layouts in HBM:
//   real grid      R[g1][g2][g3]           (g3 contiguous)
//   half spectrum  C[m3][m1][m2]           (m2 contiguous, m3 = 0 .. K3/2)
// Passes (each one read and one write of the grid, transforms in LDS):
//   1. spread + R2C along axis 3  : block = (g1, tile of TW rows g2).  The
//      atoms whose spline support reaches the tile are held in registers (one
//      per thread), their weights accumulated into the tile in 32-bit fixed
//      point with integer LDS atomics (order-independent sums; FP32 LDS
//      atomics run at a fraction of the integer rate on gfx950), converted
//      to FP32, two real rows packed into one complex FFT and the half
//      spectra written transposed so that m2 becomes contiguous.
//   2. C2C along axis 2 (rows contiguous), NR rows per block.
//   3. C2C along axis 1 (stride K2) on tiles of TW columns: forward FFT,
//      multiplication by G(m) computed on the fly, inverse FFT, in one pass.
//   4. inverse C2C along axis 2.
//   5. C2R along axis 3 back to R[g1][g2][g3].
// Every pass is a template on its axis length (and tile width, spline order):
// every supported length has fully compile-time transforms, with uniform tiles
// for the lengths of the benchmark grids and tiles of up to 16 rows for any
// axis-2 length (RAG, mesh_len.h) otherwise; the kernels with runtime sizes
// (template value 0) serve the tile widths that qeq_set_tiles asks for.
#include <math.h>

#include "mesh_len.h"
#include "mesh_passes.h"

namespace {

// ------------------------------------------------------------------ passes 1 + 2 fused
// Spread, axis-3 real-to-complex and axis-2 forward transforms of one g1
// plane in LDS, for grids whose plane half spectrum K2 (K3/2 + 1) fits (one
// block per CU): the mirror image of k_slab_inv, saving the grid round trip
// between the spread and the axis-2 pass.
//   Candidates: the atoms whose home plane h1 = g1 + k1 (k1 < p) reaches g1,
//   one index range per k1 (atoms are sorted by home bin), taken by the
//   block's threads together and held in registers (CPT per thread).
//   Fixed point, one scale per row g2: every value of row g2 is a sum of one
//   term per candidate whose axis-2 support covers the row, so |value| <=
//   S(g2) = sum of |src| w1(k1) max(w2) max(w3) over those candidates.  The
//   plane total S (< 2^eS) fixes a quantum U = 2^(eS - 20); each candidate
//   adds floor(bound / U) + 1 to the integer bounds of its p rows (integer
//   sums: order-independent), so S(g2) <= rb(g2) U, and the row is scaled by
//   2^(30 - e) with rb(g2) U < 2^e.  A row's bound sums over about p / K2 of
//   the plane's candidates (about 32 of 1,024 at 192^3 and 32,768 atoms), a
//   row tile's of k_spread_r2c over about (TW + p - 1) / K2 of them, so the
//   row scales are finer.
//   Then two real rows per complex line for the axis-3 transform (the
//   conversion inside its first radix stage), their half spectra unpacked
//   to X[g2][m3] (row stride K3/2 + 1), the axis-2 transform of NCOL m3
//   columns (at least the kept ones: 80 of 97 at 192^3 are one round of
//   radix-16 butterflies for the block, 97 two), and C[m3][g1][m2] written.
constexpr int PLANE_NT = 1024;

template <int K2C, int K3C, int NCOL>
__global__ __launch_bounds__(PLANE_NT) void k_plane_fwd(KParams k, FftAxis ax2, FftAxis ax3,
                                                       const double* __restrict__ src,
                                                       const int* __restrict__ bin_start,
                                                       const int* __restrict__ home,
                                                       const float* __restrict__ wts, float2* __restrict__ C,
                                                       const int* __restrict__ done) {
    constexpr int P = 6, CPT = 2;
    constexpr int KS = K3C / 2 + 1;   // complex row stride of X
    constexpr int AS = K3C + 1;       // int row stride of the accumulator
    constexpr int NP = K2C / 2;       // row pairs
    static_assert(K2C * AS * 4 <= K2C * KS * 8, "accumulator must fit the plane buffer");
    static_assert(K3C * NP <= K2C * KS, "packed rows must fit the plane buffer");
    extern __shared__ float2 sm[];
    float2* tw2 = sm;              // K2C: e^{-2 pi i j / K2}
    float2* tw3 = tw2 + K2C;       // K3C: e^{-2 pi i j / K3}
    float2* X = tw3 + K3C;         // K2C x KS
    int* acc = reinterpret_cast<int*>(X);
    __shared__ int rb[K2C];
    __shared__ float rinv[K2C], rsc[K2C];
    __shared__ int sh_e;
    const int tid = threadIdx.x;
    // XCD-aware plane order: the p planes that read one atom run on one XCD
    const int g1 = xcd_remap(blockIdx.x, gridDim.x);
    const int K1 = k.K1;
    // twiddles and the candidate ranges are requested before the converged
    // flag is examined, so the loads share one round trip
    constexpr int NTW = K2C + K3C;
    float2 twv = make_float2(0.f, 0.f);
    if (tid < NTW) twv = tid < K2C ? ax2.tw[tid] : ax3.tw[tid - K2C];
    int blo[P], bhi[P];
#pragma unroll
    for (int k1 = 0; k1 < P; ++k1) {
        int h1 = g1 + k1;
        if (h1 >= K1) h1 -= K1;
        blo[k1] = bin_start[h1 * K2C];
        bhi[k1] = bin_start[(h1 + 1) * K2C];
    }
    if (done && *done) return;
    if (tid < NTW) sm[tid] = twv;
    {
        int4* a4 = reinterpret_cast<int4*>(acc);
        constexpr int N4 = K2C * AS / 4;
        static_assert((K2C * AS) % 4 == 0, "accumulator clears as int4");
        for (int t = tid; t < N4; t += PLANE_NT) a4[t] = make_int4(0, 0, 0, 0);
    }
    if (tid < K2C) rb[tid] = 0;
    int off[P + 1];
    off[0] = 0;
#pragma unroll
    for (int k1 = 0; k1 < P; ++k1) off[k1 + 1] = off[k1] + (bhi[k1] - blo[k1]);
    const int ncand = off[P];
    // candidate t: plane k1 (the last range starting at or before t), atom a
    float a0[CPT], w2[CPT][P], w3[CPT][P];
    double bnd[CPT];
    int h2[CPT], h3[CPT];
    auto load = [&](int s, int t) {
        int k1 = 0, a = blo[0] + t;
#pragma unroll
        for (int u = 1; u < P; ++u) {
            if (t >= off[u]) {
                k1 = u;
                a = blo[u] + (t - off[u]);
            }
        }
        const float* w = wts + (size_t)a * 3 * QEQ_MAXP;
        const double sv = src[a];
        const float w1 = w[k1];
        a0[s] = (float)sv * w1;
        float m2 = 0.f, m3 = 0.f;
#pragma unroll
        for (int kk = 0; kk < P; ++kk) {
            w2[s][kk] = w[QEQ_MAXP + kk];
            w3[s][kk] = w[2 * QEQ_MAXP + kk];
            m2 = fmaxf(m2, w2[s][kk]);
            m3 = fmaxf(m3, w3[s][kk]);
        }
        bnd[s] = fabs((double)a0[s]) * (double)m2 * (double)m3;
        h2[s] = home[4 * a + 1];
        h3[s] = home[4 * a + 2];
    };
    const int nround = (ncand + CPT * PLANE_NT - 1) / (CPT * PLANE_NT);
    // pass A: the plane bound S (candidates of later rounds are loaded again
    // in the passes below; one round keeps them in registers)
    {
        double v[1] = {0.0};
        for (int rd = 0; rd < nround; ++rd) {
#pragma unroll
            for (int s = 0; s < CPT; ++s) {
                const int t = (rd * CPT + s) * PLANE_NT + tid;
                if (t < ncand) {
                    load(s, t);
                    v[0] += bnd[s];
                }
            }
        }
        block_sum<1>(v);   // its barriers also order the clears above
        if (tid == 0) {
            int e = 0;
            (void)frexp(v[0] > 0.0 ? v[0] : 1.0, &e);   // S < 2^e
            sh_e = e;
        }
        __syncthreads();
    }
    const int eS = sh_e;
    // pass B: integer row bounds in units of U = 2^(eS - 20); each term is
    // below 2^20 and the terms of a row sum to below 2^20 + ncand
    for (int rd = 0; rd < nround; ++rd) {
#pragma unroll
        for (int s = 0; s < CPT; ++s) {
            const int t = (rd * CPT + s) * PLANE_NT + tid;
            if (t < ncand) {
                if (nround > 1) load(s, t);
                const int q = (int)ldexp(bnd[s], 20 - eS) + 1;
#pragma unroll
                for (int k2 = 0; k2 < P; ++k2) {
                    int r = h2[s] - k2;
                    if (r < 0) r += K2C;
                    atomicAdd(rb + r, q);
                }
            }
        }
    }
    __syncthreads();
    if (tid < K2C) {
        int e = 0;
        const double sr = ldexp((double)rb[tid], eS - 20);
        (void)frexp(sr > 0.0 ? sr : 1.0, &e);   // S(g2) <= sr < 2^e
        const int x = max(-126, min(126, 30 - e));
        rsc[tid] = ldexpf(1.0f, x);
        rinv[tid] = ldexpf(1.0f, -x);
    }
    __syncthreads();
    // pass C: terms rounded to integers by one FP64 fused multiply-add with
    // 1.5 * 2^52 (the low word of the sum is the two's-complement integer)
    constexpr double RND = 6755399441055744.0;
    for (int rd = 0; rd < nround; ++rd) {
#pragma unroll
        for (int s = 0; s < CPT; ++s) {
            const int t = (rd * CPT + s) * PLANE_NT + tid;
            if (t < ncand) {
                if (nround > 1) load(s, t);
                double w3d[P];
                int col[P];
#pragma unroll
                for (int k3 = 0; k3 < P; ++k3) {
                    w3d[k3] = (double)w3[s][k3];
                    int g3 = h3[s] - k3;
                    if (g3 < 0) g3 += K3C;
                    col[k3] = g3;
                }
#pragma unroll
                for (int k2 = 0; k2 < P; ++k2) {
                    int r = h2[s] - k2;
                    if (r < 0) r += K2C;
                    const double a1 = (double)(a0[s] * rsc[r]) * (double)w2[s][k2];   // exact
                    int* row = acc + r * AS;
#pragma unroll
                    for (int k3 = 0; k3 < P; ++k3) {
                        const int v = (int)(unsigned)__double_as_longlong(fma(a1, w3d[k3], RND));
                        atomicAdd(row + col[k3], v);
                    }
                }
            }
        }
    }
    __syncthreads();
    // rows 2c and 2c + 1 as one complex line along g3 (Z[g3][c], c < NP):
    // the conversion to FP32 inside the first radix stage
    float2* Z = X;
    {
        constexpr int R0 = ct_radix_at(K3C, 0, NP, PLANE_NT), PER0 = K3C / R0;
        constexpr int ITEMS = PER0 * NP, IT0 = (ITEMS + PLANE_NT - 1) / PLANE_NT;
        float2 v[IT0][R0];
#pragma unroll
        for (int it = 0; it < IT0; ++it) {
            const int item = tid + it * PLANE_NT;
            if (ITEMS % PLANE_NT == 0 || item < ITEMS) {
                const int c = item % NP, j = item / NP;
                const int* re = acc + (2 * c) * AS;
                const int* im = re + AS;
                const float se = rinv[2 * c], so = rinv[2 * c + 1];
#pragma unroll
                for (int r = 0; r < R0; ++r) {
                    const int g3 = j + r * PER0;
                    v[it][r] = make_float2((float)re[g3] * se, (float)im[g3] * so);
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < IT0; ++it) {
            const int item = tid + it * PLANE_NT;
            if (ITEMS % PLANE_NT == 0 || item < ITEMS) {
                const int c = item % NP, j = item / NP;
                dft<R0>(v[it], false);
#pragma unroll
                for (int r = 0; r < R0; ++r) Z[(j * R0 + r) * NP + c] = v[it][r];
            }
        }
        __syncthreads();
        fft_ct<K3C, NP, NP, PLANE_NT, false, 1, R0>(Z, tw3, tid);
    }
    // unpack the two rows' half spectra, m3 = 0 .. K3/2: every LDS read of the
    // thread first (the rows overwrite the packed lines)
    {
        constexpr int NI = NP * NCOL, PI = (NI + PLANE_NT - 1) / PLANE_NT;
        float2 za[PI], zb[PI];
#pragma unroll
        for (int u = 0; u < PI; ++u) {
            const int t = tid + u * PLANE_NT;
            if (NI % PLANE_NT == 0 || t < NI) {
                const int m = t / NP, c = t - m * NP;
                za[u] = Z[m * NP + c];
                zb[u] = Z[(m == 0 ? 0 : K3C - m) * NP + c];
            }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PI; ++u) {
            const int t = tid + u * PLANE_NT;
            if (NI % PLANE_NT == 0 || t < NI) {
                const int m = t / NP, c = t - m * NP;
                const float2 Zv = za[u], Zc = make_float2(zb[u].x, -zb[u].y);
                const float2 d = csub(Zv, Zc);
                X[(2 * c) * KS + m] = make_float2(0.5f * (Zv.x + Zc.x), 0.5f * (Zv.y + Zc.y));
                X[(2 * c + 1) * KS + m] = make_float2(0.5f * d.y, -0.5f * d.x);
            }
        }
        __syncthreads();
    }
    // axis-2 transform of the first NCOL m3 columns, then C[m3][g1][m2]
    fft_ct<K2C, NCOL, KS, PLANE_NT, false>(X, tw2, tid);
    __syncthreads();
#pragma unroll 4
    for (int t = tid; t < k.K3h * K2C; t += PLANE_NT) {
        const int m3 = t / K2C, m2 = t - m3 * K2C;
        if (m2_kept(k, m2)) C[((size_t)m3 * K1 + g1) * K2C + m2] = X[m2 * KS + m3];
    }
}

// ------------------------------------------------------------------ passes 4 + 5 fused
// Inverse axis-2 and axis-3 complex-to-real transforms of one g1 slab in LDS,
// for grids whose slab half spectrum K2 (K3/2 + 1) fits (one block per CU):
//   load C[m3][g1][m2] as X[m2][m3] (row stride KS = K3/2 + 1),
//   inverse FFT along m2 for all K3/2 + 1 columns -> X[g2][m3],
//   each row g2: the real inverse DFT of length N = K3 from its half spectrum
//   as one complex inverse FFT of length N/2, in place:
//     E[k] = X[k] + conj X[N/2 - k],  O[k] = e^{2 pi i k/N} (X[k] - conj X[N/2 - k]),
//     z = IFFT_{N/2}(E + i O),  x[2n] = Re z[n],  x[2n + 1] = Im z[n]
//   (both IFFT(E) and IFFT(O) are real because the line is),
//   store R[g1][g2][g3] as pairs.  Saves the grid round trip between the two
//   separate passes.
//   INTERP: instead of storing the slab, every atom whose spline support meets
//   plane g1 (h1 = g1 + k1, k1 < p) takes its partial back-interpolation
//   w1(k1) sum_k2 w2(k2) sum_k3 w3(k3) phi(g1, h2 - k2, h3 - k3) from the slab
//   in LDS into slot 2 k1 of mpart (slot 2 k1 + 1 = 0: the whole plane is
//   here), as the fused tile pass does.
constexpr int SLAB_NT = 1024;

template <int K2C, int K3C, int NCOL, bool INTERP = false>
__global__ __launch_bounds__(SLAB_NT) void k_slab_inv(KParams k, FftAxis ax2, FftAxis ax3,
                                                     const float2* __restrict__ C, float* __restrict__ R,
                                                     const int* __restrict__ done,
                                                     const int* __restrict__ bin_start = nullptr,
                                                     const int* __restrict__ home = nullptr,
                                                     const float* __restrict__ wts = nullptr,
                                                     float* __restrict__ mpart = nullptr) {
    if (done && *done) return;
    constexpr int K3H = K3C / 2 + 1;
    constexpr int KS = K3H;
    constexpr int NH = K3C / 2;
    extern __shared__ float2 sm[];
    float2* tw2 = sm;            // K2C: e^{-2 pi i j / K2}
    float2* tw3 = tw2 + K2C;     // K3C: e^{-2 pi i j / K3}
    float2* twh = tw3 + K3C;     // NH:  e^{-2 pi i j / NH}
    float2* X = twh + NH;        // K2C x KS
    const int tid = threadIdx.x;
    // XCD-aware plane order: the p planes that read one atom's weights run
    // on the same XCD and share its L2
    const int g1 = xcd_remap(blockIdx.x, gridDim.x);
    const int K1 = k.K1;
    // interpolation: atom ranges of the p planes whose support reaches g1
    // (read now, used at the end)
    constexpr int P = 6;
    int blo[P], bhi[P];
    if constexpr (INTERP) {
#pragma unroll
        for (int k1 = 0; k1 < P; ++k1) {
            int h1 = g1 + k1;
            if (h1 >= K1) h1 -= K1;
            blo[k1] = bin_start[h1 * K2C];
            bhi[k1] = bin_start[(h1 + 1) * K2C];
        }
    }
    // The three twiddle tables (K2C + K3C + NH entries) and the plane's first
    // NCOL m3 columns (at least the kept ones; the others are zero).  All
    // columns: in two groups, the axis-2 transforms of the first running while
    // the second's loads are in flight (barriers wait on LDS only).  Fewer: in
    // one, whose radix-16 stage is then one round of the block (192^3: 80
    // columns).
    constexpr int CA = NCOL == K3H ? (K3H + 1) / 2 : NCOL, CB = NCOL - CA;
    auto ld_col = [&](int m3, int m2) {
        return m3 < k.K3h && m2_kept(k, m2) ? C[((size_t)m3 * K1 + g1) * K2C + m2] : make_float2(0.f, 0.f);
    };
    {
        auto ld_tw = [&](int t) {
            return t < K2C ? ax2.tw[t] : (t < K2C + K3C ? ax3.tw[t - K2C] : ax3.tw[2 * (t - K2C - K3C)]);
        };
        auto st_tw = [&](int t, float2 v) { tw2[t] = v; };   // tw2 | tw3 | twh are contiguous
        auto ld = [&](int t) {
            const int m3 = t / K2C, m2 = t - m3 * K2C;
            return ld_col(m3, m2);
        };
        auto st = [&](int t, float2 v) {
            const int m3 = t / K2C, m2 = t - m3 * K2C;
            X[m2 * KS + m3] = v;
        };
        stage2_ct<K2C + K3C + NH, CA * K2C, SLAB_NT, float2>(tid, ld_tw, st_tw, ld, st);
    }
    for (int t = tid; t < (K3H - NCOL) * K2C; t += SLAB_NT) {
        const int m3 = t / K2C, m2 = t - m3 * K2C;
        X[m2 * KS + NCOL + m3] = make_float2(0.f, 0.f);
    }
    constexpr int PB = (CB * K2C + SLAB_NT - 1) / SLAB_NT;
    float2 vb[PB > 0 ? PB : 1];
#pragma unroll
    for (int u = 0; u < PB; ++u) {
        const int t = tid + u * SLAB_NT;
        if ((CB * K2C) % SLAB_NT == 0 || t < CB * K2C) {
            const int m3 = t / K2C, m2 = t - m3 * K2C;
            vb[u] = ld_col(CA + m3, m2);
        }
    }
    __syncthreads();
    fft_ct<K2C, CA, KS, SLAB_NT, true>(X, tw2, tid);
    if constexpr (CB > 0) {
#pragma unroll
        for (int u = 0; u < PB; ++u) {
            const int t = tid + u * SLAB_NT;
            if ((CB * K2C) % SLAB_NT == 0 || t < CB * K2C) {
                const int m3 = t / K2C, m2 = t - m3 * K2C;
                X[m2 * KS + CA + m3] = vb[u];
            }
        }
        __syncthreads();
        fft_ct<K2C, CB, KS, SLAB_NT, true>(X + CA, tw2, tid);
    }
    // Length-NH inverse transform along each row g2 of the packed sequence
    // z(n) = (X(n) + conj X(NH - n)) + i (X(n) - conj X(NH - n)) e^{2 pi i n / K3}
    // (two real outputs per complex one).  Its first radix stage builds z
    // while loading: each item reads its R0 elements and their mirrors, so the
    // pairing costs no pass of its own over the plane.
    {
        constexpr int R0 = ct_radix_at(NH, 0, K2C, SLAB_NT);
        constexpr int PER0 = NH / R0;
        constexpr int ITEMS = PER0 * K2C;
        constexpr int IT0 = (ITEMS + SLAB_NT - 1) / SLAB_NT;
        float2 v[IT0][R0];
#pragma unroll
        for (int it = 0; it < IT0; ++it) {
            const int item = tid + it * SLAB_NT;
            if (ITEMS % SLAB_NT == 0 || item < ITEMS) {
                const int c = item % K2C, j = item / K2C;
                const float2* row = X + c * KS;
#pragma unroll
                for (int r = 0; r < R0; ++r) {
                    const int idx = j + r * PER0;
                    const float2 xk = row[idx], xq = row[NH - idx];
                    const float2 cq = make_float2(xq.x, -xq.y);
                    const float2 e = cadd(xk, cq);
                    float2 w = tw3[idx];
                    w.y = -w.y;
                    const float2 o = cmul(csub(xk, cq), w);
                    v[it][r] = make_float2(e.x - o.y, e.y + o.x);
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < IT0; ++it) {
            const int item = tid + it * SLAB_NT;
            if (ITEMS % SLAB_NT == 0 || item < ITEMS) {
                const int c = item % K2C, j = item / K2C;
                dft<R0>(v[it], true);
                float2* row = X + c * KS;
#pragma unroll
                for (int r = 0; r < R0; ++r) row[j * R0 + r] = v[it][r];
            }
        }
        __syncthreads();
        fft_ct<NH, K2C, 1, SLAB_NT, true, 1, R0, KS>(X, twh, tid);
    }
    if constexpr (!INTERP) {
        float2* R2 = reinterpret_cast<float2*>(R) + (size_t)g1 * K2C * NH;
        for (int t = tid; t < K2C * NH; t += SLAB_NT) {
            const int g2 = t / NH, n = t - g2 * NH;
            R2[t] = X[g2 * KS + n];
        }
    } else {
        // phi(g1, g2, g3) = xf[2 KS g2 + g3].  The atoms of the p planes form
        // one index range (plane k1's atoms from off[k1]), so the block's
        // threads take them all at once: one round of atom loads, not p.
        const float* xf = reinterpret_cast<const float*>(X);
        const int n = k.n;
        int off[P + 1];
        off[0] = 0;
#pragma unroll
        for (int k1 = 0; k1 < P; ++k1) off[k1 + 1] = off[k1] + (bhi[k1] - blo[k1]);
        for (int t = tid; t < off[P]; t += SLAB_NT) {
            int k1 = 0, a = blo[0] + t;
#pragma unroll
            for (int u = 1; u < P; ++u) {
                if (t >= off[u]) {
                    k1 = u;
                    a = blo[u] + (t - off[u]);
                }
            }
            {
                const float* w = wts + (size_t)a * 3 * QEQ_MAXP;
                const int h2 = home[4 * a + 1];
                const int h3 = home[4 * a + 2];
                float s = 0.f;
#pragma unroll
                for (int k2 = 0; k2 < P; ++k2) {
                    int g2 = h2 - k2;
                    if (g2 < 0) g2 += K2C;
                    const float* row = xf + 2 * KS * g2;
                    float r3 = 0.f;
#pragma unroll
                    for (int k3 = 0; k3 < P; ++k3) {
                        int g3 = h3 - k3;
                        if (g3 < 0) g3 += K3C;
                        r3 += w[2 * QEQ_MAXP + k3] * row[g3];
                    }
                    s += w[QEQ_MAXP + k2] * r3;
                }
                mpart[(size_t)(2 * k1) * n + a] = w[k1] * s;
                mpart[(size_t)(2 * k1 + 1) * n + a] = 0.f;
            }
        }
    }
}

size_t smem_spread(const KParams& k) {
    return sizeof(float2) * (size_t)k.K3 + sizeof(int) * (size_t)k.K3 * k.TWS;
}
size_t smem_rows(const KParams& k) { return sizeof(float2) * ((size_t)k.K2 + (size_t)k.K2 * (k.NR + 1)); }
size_t smem_cols(const KParams& k) { return sizeof(float2) * ((size_t)k.K1 + (size_t)k.K1 * k.TW); }
size_t smem_c2r(const KParams& k) {
    return sizeof(float2) * ((size_t)k.K3 + (size_t)(k.K3 / 2 + 1) * k.TW + (size_t)k.K3 * (k.TW / 2));
}

// Lengths with uniform tiles of their own; other lengths take the ragged tiles
// of mesh_len.h, other tile widths the runtime-sized kernels.
#define QEQ_FOR_EACH_SIZE(X) X(24, 8) X(48, 16) X(96, 16) X(192, 16) X(320, 16) X(320, 8)
#define QEQ_FOR_EACH_SPREAD(X) \
    X(24, 8) X(48, 16) X(96, 16) X(192, 12) X(192, 16) X(192, 24) X(320, 8) X(320, 16)

int spread_pass(qeq_plan* pl, const double* src, const int* done) {
    const KParams& k = pl->kp;
    dim3 g(k.K1 * k.ntile_s), b(NT);
    const size_t sh = smem_spread(k);
    ProfScope ps(pl, PK_SPREAD_R2C);
    // the accumulator of long axes can exceed the default 64 KB window
#define X(KK, TT)                                                                                  \
    if (!k.rag_s && k.K3 == KK && k.TWS == TT && k.p == 6) {                                                    \
        if (sh > 65536)                                                                            \
            QEQ_HIP(hipFuncSetAttribute((const void*)k_spread_r2c<KK, TT, 6>,                      \
                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh));     \
        hipExtLaunchKernelGGL((k_spread_r2c<KK, TT, 6>), g, b, sh, pl->stream, ps.start(), ps.stop(), 0, k, \
                              pl->axes.ax[2], src, pl->bin_start, pl->home, pl->wts, pl->grid_c, done);   \
        return qeq_check(hipGetLastError());                                                       \
    }
    QEQ_FOR_EACH_SPREAD(X)
#undef X
    if (k.rag_s) return mesh_len({pl, LEN_SPREAD, src, 0, nullptr, nullptr, nullptr, nullptr, done, ps.start(), ps.stop()}, k.K3);
    // the runtime-sized kernel indexes the tile by shifts: power-of-two widths only
    if (k.TWS & (k.TWS - 1)) return QEQ_EPLAN;
    if (sh > 65536)
        QEQ_HIP(hipFuncSetAttribute((const void*)k_spread_r2c<0, 0, 0>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)sh));
    hipExtLaunchKernelGGL((k_spread_r2c<0, 0, 0>), g, b, sh, pl->stream, ps.start(), ps.stop(), 0, k,
                          pl->axes.ax[2], src, pl->bin_start, pl->home, pl->wts, pl->grid_c, done);
    return qeq_check(hipGetLastError());
}

template <bool INV>
int rows_pass_t(qeq_plan* pl, const int* done) {
    const KParams& k = pl->kp;
    const int nrows = k.K3h * k.K1;
    dim3 g((nrows + k.NR - 1) / k.NR), b(NT);
    const size_t sh = smem_rows(k);
    ProfScope ps(pl, INV ? PK_ROWS_INV : PK_ROWS_FWD);
#define X(KK, TT)                                                                                  \
    if (k.K2 == KK && k.NR == 16) {                                                                \
        hipExtLaunchKernelGGL((k_fft_rows<KK, 16, INV>), g, b, sh, pl->stream, ps.start(), ps.stop(), 0, \
                              k, pl->axes.ax[1], pl->grid_c, nrows, done);                          \
        return qeq_check(hipGetLastError());                                                       \
    }
    QEQ_FOR_EACH_SIZE(X)
#undef X
#define X(KK)                                                                                      \
    if (k.K2 == KK && k.NR == 4) {                                                                 \
        hipExtLaunchKernelGGL((k_fft_rows<KK, 4, INV>), g, b, sh, pl->stream, ps.start(), ps.stop(), 0, \
                              k, pl->axes.ax[1], pl->grid_c, nrows, done);                          \
        return qeq_check(hipGetLastError());                                                       \
    }
    X(320)
#undef X
    if (k.NR == len_nr(k.K2))
        return mesh_len({pl, INV ? LEN_ROWS_INV : LEN_ROWS_FWD, nullptr, 0, nullptr, nullptr, nullptr, nullptr, done,
                         ps.start(), ps.stop()}, k.K2);
    hipExtLaunchKernelGGL((k_fft_rows<0, 0, INV>), g, b, sh, pl->stream, ps.start(), ps.stop(), 0, k,
                          pl->axes.ax[1], pl->grid_c, nrows, done);
    return qeq_check(hipGetLastError());
}

int rows_pass(qeq_plan* pl, int inv, const int* done) {
    return inv ? rows_pass_t<true>(pl, done) : rows_pass_t<false>(pl, done);
}

int cols_pass(qeq_plan* pl, int mode, double* epart, const int* done) {
    const KParams& k = pl->kp;
    dim3 g(k.K3h * k.ntile), b(NT);
    const size_t sh = smem_cols(k);
    ProfScope ps(pl, PK_COLS_GREEN);
    // Gaussian-on-grid densities carry no B-spline moduli
    const float* b1 = pl->pw_active ? pl->pw_ones : pl->bmod[0];
    const float* b2 = pl->pw_active ? pl->pw_ones : pl->bmod[1];
    const float* b3 = pl->pw_active ? pl->pw_ones : pl->bmod[2];
    if (k.rag) return mesh_len({pl, LEN_COLS, nullptr, mode, epart, b1, b2, b3, done, ps.start(), ps.stop()}, k.K1);
#define X(KK, TT)                                                                                  \
    if (k.K1 == KK && k.TW == TT) {                                                                \
        hipExtLaunchKernelGGL((k_fft_cols<KK, TT>), g, b, sh, pl->stream, ps.start(), ps.stop(), 0, k,   \
                              pl->axes.ax[0], pl->grid_c, b1, b2, b3, mode, epart, done);           \
        return qeq_check(hipGetLastError());                                                       \
    }
    QEQ_FOR_EACH_SIZE(X)
#undef X
    hipExtLaunchKernelGGL((k_fft_cols<0, 0>), g, b, sh, pl->stream, ps.start(), ps.stop(), 0, k, pl->axes.ax[0],
                          pl->grid_c, b1, b2, b3, mode, epart, done);
    return qeq_check(hipGetLastError());
}

int cols_virial_pass(qeq_plan* pl, double* part) {
    const KParams& k = pl->kp;
    if (k.rag)
        return mesh_len({pl, LEN_VIRIAL, nullptr, 0, part, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr}, k.K1);
    dim3 g(k.K3h * k.ntile), b(NT);
    const size_t sh = smem_cols(k);
#define X(KK, TT)                                                                                  \
    if (k.K1 == KK && k.TW == TT) {                                                                \
        hipLaunchKernelGGL((k_cols_virial<KK, TT>), g, b, sh, pl->stream, k, pl->axes.ax[0], pl->grid_c, \
                           pl->bmod[0], pl->bmod[1], pl->bmod[2], part);                            \
        return qeq_check(hipGetLastError());                                                       \
    }
    QEQ_FOR_EACH_SIZE(X)
#undef X
    hipLaunchKernelGGL((k_cols_virial<0, 0>), g, b, sh, pl->stream, k, pl->axes.ax[0], pl->grid_c, pl->bmod[0],
                       pl->bmod[1], pl->bmod[2], part);
    return qeq_check(hipGetLastError());
}

int c2r_pass(qeq_plan* pl, const int* done) {
    const KParams& k = pl->kp;
    dim3 g(k.K1 * k.ntile), b(NT);
    const size_t sh = smem_c2r(k);
    ProfScope ps(pl, PK_C2R);
    if (k.rag)
        return mesh_len({pl, LEN_C2R, nullptr, 0, nullptr, nullptr, nullptr, nullptr, done, ps.start(), ps.stop()}, k.K3);
#define X(KK, TT)                                                                                  \
    if (k.K3 == KK && k.TW == TT) {                                                                \
        hipExtLaunchKernelGGL((k_c2r<KK, TT>), g, b, sh, pl->stream, ps.start(), ps.stop(), 0, k,         \
                              pl->axes.ax[2], pl->grid_c, pl->grid_r, done);                        \
        return qeq_check(hipGetLastError());                                                       \
    }
    QEQ_FOR_EACH_SIZE(X)
#undef X
    hipExtLaunchKernelGGL((k_c2r<0, 0>), g, b, sh, pl->stream, ps.start(), ps.stop(), 0, k, pl->axes.ax[2],
                          pl->grid_c, pl->grid_r, done);
    return qeq_check(hipGetLastError());
}

// The complex-to-real pass fused with the back-interpolation (2p partials per
// atom in pl->mpart); needs TW >= p - 1 (at most two tiles per atom).
bool c2r_interp_available(const qeq_plan* pl) {
    const KParams& k = pl->kp;
    const int lo = k.rag ? len_rows_min(k.K2) : k.TW, hi = k.rag ? len_rows_max(k.K2) : k.TW;
    return pl->fused_interp && lo >= k.p - 1 && k.K2 >= hi + k.p - 1 && pl->mpart != nullptr;
}

int c2r_interp_pass(qeq_plan* pl, const int* done) {
    const KParams& k = pl->kp;
    dim3 g(k.K1 * k.ntile), b(NT);
    const size_t sh = smem_c2r(k);
    const size_t sh_ct = sizeof(float2) * ((size_t)k.K3 + (size_t)(k.K3 / 2 + 1) * k.TW);   // Z in place of X
    ProfScope ps(pl, PK_C2R);
    if (k.rag)
        return mesh_len({pl, LEN_C2R_INTERP, nullptr, 0, nullptr, nullptr, nullptr, nullptr, done, ps.start(), ps.stop()},
                        k.K3);
#define X(KK, TT)                                                                                  \
    if (k.K3 == KK && k.TW == TT && k.p == 6) {                                                     \
        hipExtLaunchKernelGGL((k_c2r_interp<KK, TT, 6>), g, b, sh_ct, pl->stream, ps.start(), ps.stop(), 0, k, \
                              pl->axes.ax[2], pl->grid_c, pl->bin_start, pl->home, pl->wts, pl->mpart, done); \
        return qeq_check(hipGetLastError());                                                       \
    }
    QEQ_FOR_EACH_SIZE(X)
#undef X
    hipExtLaunchKernelGGL((k_c2r_interp<0, 0, 0>), g, b, sh, pl->stream, ps.start(), ps.stop(), 0, k, pl->axes.ax[2],
                          pl->grid_c, pl->bin_start, pl->home, pl->wts, pl->mpart, done);
    return qeq_check(hipGetLastError());
}

size_t smem_slab(int K2, int K3) {
    return sizeof(float2) * ((size_t)K2 + K3 + K3 / 2 + (size_t)K2 * (K3 / 2 + 1));
}

// Lengths with a fused slab kernel; the slab must fit the LDS of one CU.  Third:
// the m3 columns of the narrower instance.
#define QEQ_FOR_EACH_SLAB(X) X(96, 96, 40) X(192, 192, 80)

bool slab_available(const qeq_plan* pl) {
    const KParams& k = pl->kp;
    if (!pl->fused_inverse || k.K1 < 64) return false;
#define X(A, B, N) if (k.K2 == A && k.K3 == B) return true;
    QEQ_FOR_EACH_SLAB(X)
#undef X
    return false;
}

template <int A, int B, int N, bool INTERP>
int slab_launch(qeq_plan* pl, const int* done, hipEvent_t e0, hipEvent_t e1) {
    const KParams& k = pl->kp;
    const size_t sh = smem_slab(A, B);
    QEQ_HIP(hipFuncSetAttribute((const void*)k_slab_inv<A, B, N, INTERP>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)sh));
    hipExtLaunchKernelGGL((k_slab_inv<A, B, N, INTERP>), dim3(k.K1), dim3(SLAB_NT), sh, pl->stream, e0, e1, 0, k,
                          pl->axes.ax[1], pl->axes.ax[2], pl->grid_c, pl->grid_r, done,
                          INTERP ? pl->bin_start : nullptr, INTERP ? pl->home : nullptr, INTERP ? pl->wts : nullptr,
                          INTERP ? pl->mpart : nullptr);
    return qeq_check(hipGetLastError());
}

template <bool INTERP>
int slab_pass(qeq_plan* pl, const int* done) {
    const KParams& k = pl->kp;
    ProfScope ps(pl, PK_C2R);
#define X(A, B, N)                                                                             \
    if (k.K2 == A && k.K3 == B && (!INTERP || k.p == 6)) {                                      \
        if (k.K3h <= N) return slab_launch<A, B, N, INTERP>(pl, done, ps.start(), ps.stop());   \
        return slab_launch<A, B, B / 2 + 1, INTERP>(pl, done, ps.start(), ps.stop());           \
    }
    QEQ_FOR_EACH_SLAB(X)
#undef X
    return QEQ_EPLAN;
}

int slab_interp_pass(qeq_plan* pl, const int* done) { return slab_pass<true>(pl, done); }

bool slab_interp_available(const qeq_plan* pl) {
    return slab_available(pl) && pl->fused_interp && pl->kp.p == 6 && pl->mpart != nullptr;
}

int slab_inv_pass(qeq_plan* pl, const int* done) { return slab_pass<false>(pl, done); }

// Lengths with a fused forward plane kernel (spread + axis-3 + axis-2).
#define QEQ_FOR_EACH_PLANE_FWD(X) X(192, 192, 80)

size_t smem_plane_fwd(int K2, int K3) {
    return sizeof(float2) * ((size_t)K2 + K3 + (size_t)K2 * (K3 / 2 + 1));
}

bool plane_fwd_available(const qeq_plan* pl) {
    const KParams& k = pl->kp;
    if (!pl->fused_forward || k.K1 < 64 || k.p != 6) return false;
#define X(A, B, N) if (k.K2 == A && k.K3 == B) return true;
    QEQ_FOR_EACH_PLANE_FWD(X)
#undef X
    return false;
}

template <int A, int B, int N>
int plane_fwd_launch(qeq_plan* pl, const double* src, const int* done, hipEvent_t e0, hipEvent_t e1) {
    const KParams& k = pl->kp;
    const size_t sh = smem_plane_fwd(A, B);
    QEQ_HIP(hipFuncSetAttribute((const void*)k_plane_fwd<A, B, N>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)sh));
    hipExtLaunchKernelGGL((k_plane_fwd<A, B, N>), dim3(k.K1), dim3(PLANE_NT), sh, pl->stream, e0, e1, 0, k,
                          pl->axes.ax[1], pl->axes.ax[2], src, pl->bin_start, pl->home, pl->wts, pl->grid_c, done);
    return qeq_check(hipGetLastError());
}

int plane_fwd_pass(qeq_plan* pl, const double* src, const int* done) {
    const KParams& k = pl->kp;
    ProfScope ps(pl, PK_SPREAD_R2C);
#define X(A, B, N)                                                                                  \
    if (k.K2 == A && k.K3 == B && k.p == 6) {                                                      \
        if (k.K3h <= N) return plane_fwd_launch<A, B, N>(pl, src, done, ps.start(), ps.stop());    \
        return plane_fwd_launch<A, B, B / 2 + 1>(pl, src, done, ps.start(), ps.stop());            \
    }
    QEQ_FOR_EACH_PLANE_FWD(X)
#undef X
    return QEQ_EPLAN;
}

// Forward axis-2, axis-1 with the Green's function, inverse axis-2: one pass
// where the planes fit.
int middle(qeq_plan* pl, bool fwd, bool inv, const int* done) {
    if (fwd && inv && mid_available(pl)) {
        ProfScope ps(pl, PK_COLS_GREEN);
        const bool pw = pl->pw_active;
        return launch_mid(pl, pw ? pl->pw_ones : pl->bmod[0], pw ? pl->pw_ones : pl->bmod[1],
                          pw ? pl->pw_ones : pl->bmod[2], done, ps.start(), ps.stop());
    }
    if (fwd) QEQ_TRY(rows_pass(pl, 0, done));
    QEQ_TRY(cols_pass(pl, MESH_FWD | MESH_GREEN | MESH_INV, nullptr, done));
    return inv ? rows_pass(pl, 1, done) : QEQ_OK;
}

// From the axis-3 half spectrum to the potential: the axis-2 transforms are
// left out where the fused plane kernel (forward) did, or the fused slab kernel
// (inverse) does them.
int after_axis3(qeq_plan* pl, bool fwd, const int* done) {
    const bool slab = slab_available(pl);
    QEQ_TRY(middle(pl, fwd, !slab, done));
    return slab ? slab_inv_pass(pl, done) : c2r_pass(pl, done);
}

// Spread, axis-3 and, with the plane kernel, axis-2 transform.
int forward_head(qeq_plan* pl, const double* src, const int* done) {
    return plane_fwd_available(pl) ? plane_fwd_pass(pl, src, done) : spread_pass(pl, src, done);
}

}  // namespace

bool spread_tile_compiled(int K3, int tws, int p) {
#define X(KK, TT) if (K3 == KK && tws == TT && p == 6) return true;
    QEQ_FOR_EACH_SPREAD(X)
#undef X
    return false;
}

bool rows_compiled(int K2, int nr) {
#define X(KK, TT) if (K2 == KK && nr == 16) return true;
    QEQ_FOR_EACH_SIZE(X)
#undef X
    return K2 == 320 && nr == 4;
}

bool mesh_tile_compiled(int K1, int K3, int tw, int p) {
    bool a = false, c = false;
#define X(KK, TT)                          \
    a = a || (K1 == KK && tw == TT);       \
    c = c || (K3 == KK && tw == TT);
    QEQ_FOR_EACH_SIZE(X)
#undef X
    return a && c && p == 6;
}

size_t qeq_mesh_max_smem(const KParams& k) {
    size_t a = smem_spread(k), b = smem_rows(k), c = smem_cols(k), d = smem_c2r(k);
    size_t m = a > b ? a : b;
    m = m > c ? m : c;
    return m > d ? m : d;
}

int launch_mesh_potential(qeq_plan* pl, const double* src, const int* done) {
    QEQ_TRY(forward_head(pl, src, done));
    return after_axis3(pl, !plane_fwd_available(pl), done);
}

int launch_mesh_cg(qeq_plan* pl, const double* src, const int* done, bool* partials) {
    *partials = false;
    const bool slab = slab_interp_available(pl);
    if (!slab && !c2r_interp_available(pl)) return launch_mesh_potential(pl, src, done);
    QEQ_TRY(forward_head(pl, src, done));
    QEQ_TRY(middle(pl, !plane_fwd_available(pl), !slab, done));
    *partials = true;
    return slab ? slab_interp_pass(pl, done) : c2r_interp_pass(pl, done);
}

int launch_mesh_r2c(qeq_plan* pl, const int* done) {
    return mesh_len({pl, LEN_R2C, nullptr, 0, nullptr, nullptr, nullptr, nullptr, done, nullptr, nullptr}, pl->kp.K3);
}

int launch_mesh_from_spectrum(qeq_plan* pl, const int* done) { return after_axis3(pl, true, done); }

// One pass on its own (for timing): the spread, or the complex-to-real pass
// that the CG products run (interpolating from LDS where they do).
int launch_mesh_stage(qeq_plan* pl, int kind, const double* src) {
    if (kind == PK_SPREAD_R2C)
        return plane_fwd_available(pl) ? plane_fwd_pass(pl, src, nullptr) : spread_pass(pl, src, nullptr);
    if (kind == PK_C2R) {
        if (slab_interp_available(pl)) return slab_interp_pass(pl, nullptr);
        if (c2r_interp_available(pl)) return c2r_interp_pass(pl, nullptr);
        return slab_available(pl) ? slab_inv_pass(pl, nullptr) : c2r_pass(pl, nullptr);
    }
    return QEQ_EINVAL;
}

int mesh_virial_blocks(const KParams& k) { return k.K3h * k.ntile; }

int launch_mesh_virial(qeq_plan* pl, const double* src, double* part) {
    QEQ_TRY(spread_pass(pl, src, nullptr));
    QEQ_TRY(rows_pass(pl, 0, nullptr));
    return cols_virial_pass(pl, part);
}
