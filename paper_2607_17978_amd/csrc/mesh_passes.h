// Mesh passes of one axis length each (templates): see mesh.hip for the
// layouts and the order of the passes.
#pragma once

#include <math.h>

#include "internal.h"

namespace {

#define MESH_FWD 1
#define MESH_GREEN 2
#define MESH_INV 4
#define MESH_ENERGY 8

constexpr int NT = QEQ_FFT_THREADS;

__device__ __forceinline__ int ilog2_dev(int x) { return 31 - __clz(x); }

// Whether the passes carry index m2 (KParams::M2).
__device__ __forceinline__ bool m2_kept(const KParams& k, int m2) { return m2 <= k.M2 || m2 >= k.K2 - k.M2; }

// First row and row count of axis-2 tile t.  Uniform tiles of TW rows, or
// (RAG) ntile tiles of an even number of rows, at most TW, as equal as
// possible: any axis-2 length, no tile much narrower than the others (an
// atom's p rows meet at most two of them).
template <bool RAG>
__device__ __forceinline__ void tile_of(int t, int ntile, int K2, int TW, int& g20, int& W) {
    if (RAG) {
        const int np = K2 >> 1;
        const int a = t * np / ntile, b = (t + 1) * np / ntile;
        g20 = 2 * a;
        W = 2 * (b - a);
    } else {
        g20 = t * TW;
        W = TW;
    }
}

// ------------------------------------------------------------------ pass 1
template <int KC, int TWC, int PC, bool RAG = false>
__global__ __launch_bounds__(NT) void k_spread_r2c(KParams k, FftAxis ax3, const double* __restrict__ src,
                                                  const int* __restrict__ bin_start,
                                                  const int* __restrict__ home,
                                                  const float* __restrict__ wts, float2* __restrict__ C,
                                                  const int* __restrict__ done) {
    extern __shared__ float2 sm[];
    const int K3 = KC ? KC : k.K3;
    const int TW = TWC ? TWC : k.TWS;
    const int p = PC ? PC : k.p;
    const int ncol = TW >> 1;
    // LDS: twiddles | accumulator acc[g3][row] (int32; the FFT buffer
    // buf[g3][pr] (complex, two rows per element) takes its place once
    // converted)
    float2* tw = sm;
    int* acc = reinterpret_cast<int*>(sm + K3);
    float2* buf = sm + K3;
    __shared__ int seg_lo[2 * QEQ_MAXP], seg_off[2 * QEQ_MAXP + 1], seg_k1[2 * QEQ_MAXP];
    __shared__ int seg_len[2 * QEQ_MAXP];
    __shared__ float sh_scale;
    const int tid = threadIdx.x;
    const int blk = xcd_remap(blockIdx.x, gridDim.x);
    const int g1 = blk / k.ntile_s;
    const int K1 = k.K1, K2 = k.K2;
    int g20, W;
    tile_of<RAG>(blk - g1 * k.ntile_s, k.ntile_s, K2, TW, g20, W);

    // The twiddles and the candidate bin bounds are requested before the
    // converged flag is examined, so the three loads share one round trip.
    // Candidate segments: for each k1, homes h1 = g1 + k1 and h2 in
    // [g20, g20 + TW + p - 1) (two pieces when the h2 range wraps); lanes
    // k1 < p fetch their bounds.
    constexpr bool TW1 = KC > 0;
    constexpr int PT = KC > 0 ? (KC + NT - 1) / NT : 1;
    float2 twv[PT];
#pragma unroll
    for (int u = 0; u < PT; ++u)
        if (TW1 && tid + u * NT < K3) twv[u] = ax3.tw[tid + u * NT];
    int lo0 = 0, len0 = 0, lo1 = 0, len1 = 0;
    if (tid < p) {
        int h1 = g1 + tid;
        if (h1 >= K1) h1 -= K1;
        const int b0 = h1 * K2;
        const int hi = g20 + W + p - 1;
        const int e1 = hi < K2 ? hi : K2;
        lo0 = bin_start[b0 + g20];
        len0 = bin_start[b0 + e1];
        if (hi > K2) {
            lo1 = bin_start[b0];
            len1 = bin_start[b0 + (hi - K2)];
        }
    }
    if (done && *done) return;
    if (TW1) {
#pragma unroll
        for (int u = 0; u < PT; ++u)
            if (tid + u * NT < K3) tw[tid + u * NT] = twv[u];
    } else {
        for (int t = tid; t < K3; t += NT) tw[t] = ax3.tw[t];
    }
    for (int t = tid; t < K3 * TW; t += NT) acc[t] = 0;
    if (tid < p) {
        seg_lo[2 * tid] = lo0;
        seg_len[2 * tid] = len0 - lo0;
        seg_lo[2 * tid + 1] = lo1;
        seg_len[2 * tid + 1] = len1 - lo1;
        seg_k1[2 * tid] = tid;
        seg_k1[2 * tid + 1] = tid;
    }
    __syncthreads();
    if (tid == 0) {
        int off = 0;
        for (int sg = 0; sg < 2 * p; ++sg) {
            seg_off[sg] = off;
            off += seg_len[sg];
        }
        seg_off[2 * p] = off;
    }
    __syncthreads();
    const int ncand = seg_off[2 * p];
    // Candidate c of a round is held by thread c in registers: its
    // source value times the axis-1 weight, the axis-2 and axis-3 weights and
    // its home indices (no LDS staging, so more blocks fit per CU).
    constexpr int PM = PC ? PC : QEQ_MAXP;
    float a0 = 0.f, w2[PM], w3[PM];
    int h2 = 0, h3 = 0;
    double abound = 0.0;
    auto seg_of = [&](int cidx) {
        // last segment starting at or before cidx (empty segments share their
        // start with the next one and are passed over); independent LDS reads
        int sg = 0;
#pragma unroll
        for (int s2 = 1; s2 < 2 * PM; ++s2) {
            if (!PC && s2 >= 2 * p) break;
            sg += cidx >= seg_off[s2] ? 1 : 0;
        }
        return sg;
    };
    auto load_cand = [&](int cidx) {
        const int sg = seg_of(cidx);
        const int a = seg_lo[sg] + (cidx - seg_off[sg]);
        const float* w = wts + (size_t)a * 3 * QEQ_MAXP;
        const double sv = src[a];
        const float w1 = w[seg_k1[sg]];
        a0 = (float)sv * w1;
        float m2 = 0.f, m3 = 0.f;
#pragma unroll
        for (int kk = 0; kk < PM; ++kk) {
            if (!PC && kk >= p) break;
            w2[kk] = w[QEQ_MAXP + kk];
            w3[kk] = w[2 * QEQ_MAXP + kk];
            m2 = fmaxf(m2, w2[kk]);
            m3 = fmaxf(m3, w3[kk]);
        }
        abound = fabs(sv) * (double)w1 * (double)m2 * (double)m3;
        h2 = home[4 * a + 1];
        h3 = home[4 * a + 2];
    };
    // Fixed-point scale: every grid value of the tile is a sum over the
    // candidates of one term each, src w1(k1) w2(k2) w3(k3), so |value| <=
    // S = sum over candidates of |src| w1 max(w2) max(w3); with scale =
    // 2^(30 - e), S < 2^e, every scaled term and partial sum (rounding of
    // each term included) stays below 2^31 in magnitude.  The step 2^(e-30)
    // is at most 2^-29 S: with the weight maxima in S, about the rounding
    // of the FP32 transforms that follow.  One round: S from the registers;
    // more rounds: a pass over the candidates first.
    const bool one_round = ncand <= NT;
    {
        double v[1] = {0.0};
        if (one_round) {
            if (tid < ncand) {
                load_cand(tid);
                v[0] = abound;
            }
        } else {
            for (int cidx = tid; cidx < ncand; cidx += NT) {
                load_cand(cidx);
                v[0] += abound;
            }
        }
        block_sum<1>(v);
        if (tid == 0) {
            int e = 0;
            (void)frexp(v[0] > 0.0 ? v[0] : 1.0, &e);   // v < 2^e
            sh_scale = ldexpf(1.0f, max(-126, min(126, 30 - e)));
        }
        __syncthreads();
    }
    const float scale = sh_scale;
    // A term t (|t| < 2^31) becomes an integer by one FP64 fused multiply-add
    // with 1.5 * 2^52: the sum lies in [2^52, 2^53), where the spacing of
    // doubles is 1, so it is t rounded to the nearest integer plus 2^52 + 2^51,
    // and the low word of its bit pattern (that of 1.5 * 2^52 is zero) is the
    // two's-complement integer.
    constexpr double RND = 6755399441055744.0;   // 1.5 * 2^52
    for (int base = 0; base < ncand; base += NT) {
        const int cidx = base + tid;
        if (cidx < ncand) {
            if (!one_round) load_cand(cidx);
            const double as = (double)(a0 * scale);
            double w3d[PM];
            int col[PM];
#pragma unroll
            for (int k3 = 0; k3 < PM; ++k3) {
                if (!PC && k3 >= p) break;
                w3d[k3] = (double)w3[k3];
                int g3 = h3 - k3;
                if (g3 < 0) g3 += K3;
                col[k3] = g3 * TW;
            }
#pragma unroll
            for (int k2 = 0; k2 < PM; ++k2) {
                if (!PC && k2 >= p) break;
                // row of grid point h2 - k2 inside this tile; a tile narrower
                // than p - 1 rows also sees candidates whose point lies before it
                int r = h2 - k2 - g20;
                if (r < 0) r += K2;
                if (r < 0 || r >= W) continue;
                const double a1 = as * (double)w2[k2];   // exact: two 24-bit significands
#pragma unroll
                for (int k3 = 0; k3 < PM; ++k3) {
                    if (!PC && k3 >= p) break;
                    const int t = (int)(unsigned)__double_as_longlong(fma(a1, w3d[k3], RND));
                    atomicAdd(acc + col[k3] + r, t);
                }
            }
        }
    }
    __syncthreads();
    // fixed point -> FP32, packed two real rows per complex column, then the
    // axis-3 transform
    const float inv = 1.0f / scale;
    if constexpr (KC > 0 && TWC > 0) {
        // the conversion happens inside the first radix stage: each item
        // reads the fixed-point values of its R0 inputs into registers, and
        // after the barrier the stage's outputs overwrite the accumulator
        constexpr int NCS = TWC / 2;
        constexpr int R0 = ct_radix_at(KC, 0, NCS, NT), PER0 = KC / R0;
        constexpr int ITEMS = PER0 * NCS, IT0 = (ITEMS + NT - 1) / NT;
        float2 v[IT0][R0];
#pragma unroll
        for (int it = 0; it < IT0; ++it) {
            const int item = tid + it * NT;
            if (ITEMS % NT == 0 || item < ITEMS) {
                const int c = item % NCS, j = item / NCS;
#pragma unroll
                for (int r = 0; r < R0; ++r) {
                    const int2 a = *reinterpret_cast<const int2*>(acc + (j + r * PER0) * TWC + 2 * c);
                    v[it][r] = make_float2((float)a.x * inv, (float)a.y * inv);
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < IT0; ++it) {
            const int item = tid + it * NT;
            if (ITEMS % NT == 0 || item < ITEMS) {
                const int c = item % NCS, j = item / NCS;
                dft<R0>(v[it], false);
#pragma unroll
                for (int r = 0; r < R0; ++r) buf[(j * R0 + r) * NCS + c] = v[it][r];
            }
        }
        __syncthreads();
        fft_ct<KC, NCS, NCS, NT, false, 1, R0>(buf, tw, tid);
    } else {
        // runtime sizes: convert through registers one chunk of NT at a time
        for (int e0 = 0; e0 < K3 * ncol; e0 += NT) {
            const int e = e0 + tid;
            float2 v = make_float2(0.f, 0.f);
            if (e < K3 * ncol) {
                const int g3 = e / ncol, pr = e - g3 * ncol;
                v = make_float2((float)acc[g3 * TW + 2 * pr] * inv, (float)acc[g3 * TW + 2 * pr + 1] * inv);
            }
            __syncthreads();
            if (e < K3 * ncol) buf[e] = v;
            __syncthreads();
        }
        __syncthreads();
        fft_lds(buf, ax3, ilog2_dev(ncol), tw, false, tid, NT);
    }
    // unpack the two real rows of each complex column and write the half spectra
    const int K3h = k.K3h;
    if constexpr (KC > 0 && TWC > 0) {
        // compile-time tiles: every LDS read of the thread first, then the
        // unpacking (both rows' formulas, selected) and the stores
        constexpr int NW = (KC / 2 + 1) * TWC, PW = (NW + NT - 1) / NT, NCS = TWC / 2;
        float2 zv[PW], zc[PW];
#pragma unroll
        for (int u = 0; u < PW; ++u) {
            const int t = tid + u * NT;
            if (NW % NT == 0 || t < NW) {
                const int m = t / TWC, pr = (t - m * TWC) >> 1;
                if (m >= k.K3h) break;   // planes that are not kept
                zv[u] = buf[m * NCS + pr];
                zc[u] = buf[(m == 0 ? 0 : KC - m) * NCS + pr];
            }
        }
#pragma unroll
        for (int u = 0; u < PW; ++u) {
            const int t = tid + u * NT;
            if (NW % NT == 0 || t < NW) {
                const int m = t / TWC, r = t - m * TWC;
                if (m >= k.K3h) break;
                const float2 Z = zv[u], Zc = make_float2(zc[u].x, -zc[u].y);
                const float2 ev = make_float2(0.5f * (Z.x + Zc.x), 0.5f * (Z.y + Zc.y));
                const float2 d = csub(Z, Zc);
                const float2 od = make_float2(0.5f * d.y, -0.5f * d.x);
                if (!RAG || r < W) C[((size_t)m * K1 + g1) * K2 + g20 + r] = (r & 1) ? od : ev;
            }
        }
        return;
    }
    const int twl = ilog2_dev(TW);
    for (int t = tid; t < K3h * TW; t += NT) {
        // compile-time tiles may have any even width (division by a constant)
        const int m = TWC ? t / TWC : t >> twl;
        const int r = t - m * TW;
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

// Pass 1 for a density that is already on the real grid (the Gaussian-on-grid
// operator): real-to-complex along axis 3 of a (g1, row tile), two real rows per
// complex line, as the spread's second half.  TWC is the widest tile.
template <int KC, int TWC>
__global__ __launch_bounds__(NT) void k_r2c(KParams k, FftAxis ax3, const float* __restrict__ R,
                                           float2* __restrict__ C, const int* __restrict__ done) {
    if (done && *done) return;
    extern __shared__ float2 sm[];
    float2* tw = sm;
    float2* buf = sm + KC;
    float* acc = reinterpret_cast<float*>(buf);   // [g3][row]
    const int tid = threadIdx.x;
    const int K1 = k.K1, K2 = k.K2;
    const int blk = xcd_remap(blockIdx.x, gridDim.x);
    const int g1 = blk / k.ntile;
    int g20, W;
    tile_of<true>(blk - g1 * k.ntile, k.ntile, K2, TWC, g20, W);
    constexpr int NCS = TWC / 2, N4 = TWC * (KC / 4);
    // lanes: 16 rows times 4 pieces of 16 bytes
    stage2_ct<KC, N4, NT, float4>(
        tid, [&](int t) { const float2 w = ax3.tw[t]; return make_float4(w.x, w.y, 0.f, 0.f); },
        [&](int t, float4 v) { tw[t] = make_float2(v.x, v.y); },
        [&](int t) {
            const int r = t % TWC, c4 = t / TWC;
            return r < W ? *reinterpret_cast<const float4*>(R + ((size_t)g1 * K2 + g20 + r) * KC + 4 * c4)
                         : make_float4(0.f, 0.f, 0.f, 0.f);
        },
        [&](int t, float4 v) {
            const int r = t % TWC, c4 = t / TWC;
            acc[(4 * c4) * TWC + r] = v.x;
            acc[(4 * c4 + 1) * TWC + r] = v.y;
            acc[(4 * c4 + 2) * TWC + r] = v.z;
            acc[(4 * c4 + 3) * TWC + r] = v.w;
        });
    __syncthreads();
    fft_ct<KC, NCS, NCS, NT, false>(buf, tw, tid);
    constexpr int NW = (KC / 2 + 1) * TWC, PW = (NW + NT - 1) / NT;
#pragma unroll
    for (int u = 0; u < PW; ++u) {
        const int t = tid + u * NT;
        if (NW % NT == 0 || t < NW) {
            const int m = t / TWC, r = t - m * TWC, pr = r >> 1;
            if (m >= k.K3h || r >= W) continue;
            const float2 Z = buf[m * NCS + pr];
            float2 Zc = buf[(m == 0 ? 0 : KC - m) * NCS + pr];
            Zc.y = -Zc.y;
            const float2 ev = make_float2(0.5f * (Z.x + Zc.x), 0.5f * (Z.y + Zc.y));
            const float2 d = csub(Z, Zc);
            const float2 od = make_float2(0.5f * d.y, -0.5f * d.x);
            C[((size_t)m * K1 + g1) * K2 + g20 + r] = (r & 1) ? od : ev;
        }
    }
}

// ------------------------------------------------------------------ passes 2 / 4
// LDS layout [k][row] with row stride NR + 1 (odd) for the compile-time path,
// which keeps the transposing loads and stores free of bank conflicts.
template <int KC, int NRC, bool INV>
__global__ __launch_bounds__(NT) void k_fft_rows(KParams k, FftAxis ax2, float2* __restrict__ C, int nrows,
                                                const int* __restrict__ done) {
    if (done && *done) return;
    extern __shared__ float2 sm[];
    const int K2 = KC ? KC : k.K2;
    const int NR = NRC ? NRC : k.NR;
    const int KS = NRC ? NRC + 1 : NR;
    float2* tw = sm;
    float2* buf = sm + K2;
    const int tid = threadIdx.x;
    const int row0 = blockIdx.x * NR;
    auto ld_tw = [&](int t) { return ax2.tw[t]; };
    auto st_tw = [&](int t, float2 v) { tw[t] = v; };
    auto ld = [&](int t) {
        const int row = t / K2, kk = t - row * K2;
        return (row0 + row < nrows && (!INV || m2_kept(k, kk))) ? C[(size_t)(row0 + row) * K2 + kk]
                                                                 : make_float2(0.f, 0.f);
    };
    auto st = [&](int t, float2 v) {
        const int row = t / K2, kk = t - row * K2;
        buf[kk * KS + row] = v;
    };
    if constexpr (KC > 0 && NRC > 0) {
        stage2_ct<KC, NRC * KC, NT, float2>(tid, ld_tw, st_tw, ld, st);
    } else {
        stage_rt<4, float2>(K2, tid, NT, ld_tw, st_tw);
        stage_rt<4, float2>(NR * K2, tid, NT, ld, st);
    }
    __syncthreads();
    if constexpr (KC > 0 && NRC > 0)
        fft_ct<KC, NRC, NRC + 1, NT, INV>(buf, tw, tid);
    else
        fft_lds(buf, ax2, k.NRlog2, tw, INV, tid, NT);
    auto ld_out = [&](int t) {
        const int row = t / K2, kk = t - row * K2;
        return buf[kk * KS + row];
    };
    auto st_out = [&](int t, float2 v) {
        const int row = t / K2, kk = t - row * K2;
        if (row0 + row < nrows && (INV || m2_kept(k, kk))) C[(size_t)(row0 + row) * K2 + kk] = v;
    };
    if constexpr (KC > 0 && NRC > 0)
        stage_ct<NRC * KC, NT, float2>(tid, ld_out, st_out);   // LDS reads first, then the stores
    else
        stage_rt<4, float2>(NR * K2, tid, NT, ld_out, st_out);
}

// Reciprocal kernel of the split (SI "Ewald Summation" Gaussian filter with the
// eq. matvec Poisson kernel 4 pi / k^2), times the B-spline moduli |b_a|^2:
//   G(m) = (4 pi / V) exp(-eta^2 k^2 / 2) / k^2 |b_1(m_1)|^2 |b_2(m_2)|^2 |b_3(m_3)|^2,
// k = 2 pi H^{-1} m; G = 0 at m = 0 and on the Nyquist planes (where the
// half-spectrum symmetry of a triclinic cell is ambiguous; the Gaussian there
// is below 1e-14 for grids at the supported spacings).  Evaluated in FP32: it
// multiplies an FP32 spectrum, and FP32 exp / divide keep its relative error
// at a few ulp.
__device__ __forceinline__ float green_core(const KParams& k, int m1, int m2, int m3) {
    if ((m1 | m2 | m3) == 0) return 0.f;
    if (2 * m1 == k.K1 || 2 * m2 == k.K2 || 2 * m3 == k.K3) return 0.f;
    const float x1 = (float)(m1 <= k.K1 / 2 ? m1 : m1 - k.K1);
    const float x2 = (float)(m2 <= k.K2 / 2 ? m2 : m2 - k.K2);
    const float x3 = (float)m3;
    const float q = (float)k.M[0] * x1 * x1 + (float)k.M[1] * x2 * x2 + (float)k.M[2] * x3 * x3 +
                    2.0f * ((float)k.M[3] * x1 * x2 + (float)k.M[4] * x1 * x3 + (float)k.M[5] * x2 * x3);
    const float k2 = 39.478417604357434475f * q;   // (2 pi)^2
    const float eta = (float)k.eta_green;
    return (float)k.green_pref * expf(-0.5f * eta * eta * k2) / k2;
}

__device__ __forceinline__ float green_value(const KParams& k, int m1, int m2, int m3,
                                             const float* __restrict__ b1, const float* __restrict__ b2,
                                             const float* __restrict__ b3) {
    const float g = green_core(k, m1, m2, m3);
    return g * b1[m1] * b2[m2] * b3[m3];
}

// ------------------------------------------------------------------ pass 3
template <int KC, int TWC, bool RAG = false>
__global__ __launch_bounds__(NT) void k_fft_cols(KParams k, FftAxis ax1, float2* __restrict__ C,
                                                const float* __restrict__ b1, const float* __restrict__ b2,
                                                const float* __restrict__ b3, int mode,
                                                double* __restrict__ epart, const int* __restrict__ done) {
    if (done && *done) return;
    extern __shared__ float2 sm[];
    const int K1 = KC ? KC : k.K1;
    const int TW = TWC ? TWC : k.TW;
    const int twl = ilog2_dev(TW);
    float2* tw = sm;
    float2* buf = sm + K1;
    const int tid = threadIdx.x;
    const int K2 = k.K2;
    const int m3 = blockIdx.x / k.ntile;
    int g20, W;
    tile_of<RAG>(blockIdx.x - m3 * k.ntile, k.ntile, K2, TW, g20, W);
    if (!m2_kept(k, g20) && !m2_kept(k, g20 + W - 1)) return;   // no column of the tile is kept
    float2* base = C + (size_t)m3 * K1 * K2 + g20;
    constexpr bool CT = KC > 0 && TWC > 0;
    if constexpr (CT) {
        if ((mode & (MESH_FWD | MESH_GREEN | MESH_INV)) == (MESH_FWD | MESH_GREEN | MESH_INV)) {
            // The full product pass with the global-memory traffic folded into
            // the transforms: the forward transform's first radix stage reads
            // its inputs from HBM, the Green's function multiplies the inverse
            // transform's first-stage inputs as they are read, and the
            // inverse transform's last stage stores straight to HBM; each
            // saves an LDS pass and a barrier.  Every item of every stage
            // keeps the thread's column c = tid mod TW (NT is a multiple of
            // TW), so the Green's function's m2 is fixed per thread.
            constexpr int R0 = ct_radix_at(KC, 0, TWC, NT), PER0 = KC / R0;
            constexpr int IT0 = (PER0 * TWC + NT - 1) / NT;
            constexpr int NST = ct_nstages(KC, TWC, NT);
            static_assert(NST >= 2, "the first and the last stage are distinct");
            constexpr int RL = ct_radix_at(KC, NST - 1, TWC, NT), NSL = ct_span(KC, NST - 1, TWC, NT), PERL = KC / RL;
            constexpr int ITL = (PERL * TWC + NT - 1) / NT;
            constexpr int PT = (KC + NT - 1) / NT;
            const int c = tid & (TWC - 1);
            const bool live = (!RAG || c < W) && m2_kept(k, g20 + c);
            const int m2 = live ? g20 + c : g20;
            float2 twv[PT], v[IT0][R0];
            float bmv[IT0][R0];
            // twiddles, the tile and the moduli of the thread's elements, all
            // requested before any is used
#pragma unroll
            for (int u = 0; u < PT; ++u)
                if (tid + u * NT < KC) twv[u] = ax1.tw[tid + u * NT];
#pragma unroll
            for (int it = 0; it < IT0; ++it) {
                const int item = tid + it * NT;
                if ((PER0 * TWC) % NT == 0 || item < PER0 * TWC) {
                    const int j = item / TWC;
#pragma unroll
                    for (int r = 0; r < R0; ++r) {
                        const int g1 = j + r * PER0;
                        v[it][r] = live ? base[(size_t)g1 * K2 + c] : make_float2(0.f, 0.f);
                        bmv[it][r] = b1[g1];   // index of the same element after the transform
                    }
                }
            }
            const float bm23v = b2[m2] * b3[m3];
#pragma unroll
            for (int u = 0; u < PT; ++u)
                if (tid + u * NT < KC) tw[tid + u * NT] = twv[u];
            // forward transform: first stage from registers (no twiddles), the rest in LDS
#pragma unroll
            for (int it = 0; it < IT0; ++it) {
                const int item = tid + it * NT;
                if ((PER0 * TWC) % NT == 0 || item < PER0 * TWC) {
                    const int j = item / TWC;
                    dft<R0>(v[it], false);
#pragma unroll
                    for (int r = 0; r < R0; ++r) buf[(j * R0 + r) * TWC + c] = v[it][r];
                }
            }
            __syncthreads();
            fft_ct<KC, TWC, TWC, NT, false, 1, R0>(buf, tw, tid);
            // Green's function on the inverse transform's first-stage inputs
            // (the quadratic form k^2 / (2 pi)^2 = M11 x1^2 + l1 x1 + q23,
            // hardware exp2 and reciprocal)
            const float x2 = (float)(m2 <= k.K2 / 2 ? m2 : m2 - k.K2), x3 = (float)m3;
            const float M11 = (float)k.M[0];
            const float l1 = 2.0f * ((float)k.M[3] * x2 + (float)k.M[4] * x3);
            const float q23 = (float)k.M[1] * x2 * x2 + (float)k.M[2] * x3 * x3 + 2.0f * (float)k.M[5] * x2 * x3;
            const float eta = (float)k.eta_green;
            const float ce = -0.5f * eta * eta * 39.478417604357434475f * 1.4426950408889634f;
            const float pref = (float)k.green_pref / 39.478417604357434475f;
            const bool nyq23 = 2 * m2 == k.K2 || 2 * m3 == k.K3;
            const float mult = (m3 == 0) ? 1.f : 2.f;
            double e = 0.0;
#pragma unroll
            for (int it = 0; it < IT0; ++it) {
                const int item = tid + it * NT;
                if ((PER0 * TWC) % NT == 0 || item < PER0 * TWC) {
                    const int j = item / TWC;
#pragma unroll
                    for (int r = 0; r < R0; ++r) {
                        const int m1 = j + r * PER0;
                        const float x1 = (float)(m1 <= KC / 2 ? m1 : m1 - KC);
                        const float q = fmaf(fmaf(M11, x1, l1), x1, q23);
                        float g = pref * __builtin_amdgcn_exp2f(ce * q) * __builtin_amdgcn_rcpf(q) *
                                  (bmv[it][r] * bm23v);
                        if (nyq23 || 2 * m1 == KC || (m1 | m2 | m3) == 0) g = 0.f;
                        const float2 x = buf[m1 * TWC + c];
                        if (mode & MESH_ENERGY) e += (double)(g * mult * (x.x * x.x + x.y * x.y));
                        v[it][r] = make_float2(x.x * g, x.y * g);
                    }
                }
            }
            if (mode & MESH_ENERGY) {
                double ev[1] = {e};
                block_sum<1>(ev);
                if (tid == 0) epart[blockIdx.x] = ev[0];
            }
            __syncthreads();
#pragma unroll
            for (int it = 0; it < IT0; ++it) {
                const int item = tid + it * NT;
                if ((PER0 * TWC) % NT == 0 || item < PER0 * TWC) {
                    const int j = item / TWC;
                    dft<R0>(v[it], true);
#pragma unroll
                    for (int r = 0; r < R0; ++r) buf[(j * R0 + r) * TWC + c] = v[it][r];
                }
            }
            __syncthreads();
            fft_ct<KC, TWC, TWC, NT, true, 1, R0, 1, NST - 1>(buf, tw, tid);
            // last inverse stage: LDS to registers, twiddles, DFT, stores to HBM
            constexpr int STEPL = KC / (NSL * RL);
#pragma unroll
            for (int it = 0; it < ITL; ++it) {
                const int item = tid + it * NT;
                if ((PERL * TWC) % NT == 0 || item < PERL * TWC) {
                    const int j = item / TWC;
                    float2 u[RL];
#pragma unroll
                    for (int r = 0; r < RL; ++r) u[r] = buf[(j + r * PERL) * TWC + c];
                    const int kk = j % NSL;
#pragma unroll
                    for (int r = 1; r < RL; ++r) {
                        float2 w = tw[kk * r * STEPL];
                        w.y = -w.y;
                        u[r] = cmul(u[r], w);
                    }
                    dft<RL>(u, true);
                    const int bk = (j - kk) * RL + kk;
#pragma unroll
                    for (int r = 0; r < RL; ++r)
                        if (live) base[(size_t)(bk + r * NSL) * K2 + c] = u[r];
                }
            }
            return;
        }
    }
    // compile-time tiles: the B-spline moduli of the Green's function are
    // loaded with the tile (a thread's column c = t mod TW is the same for all
    // its elements, since NT is a multiple of TW)
    constexpr int PER = CT ? (KC * TWC + NT - 1) / NT : 1;
    float bm1[PER];
    float bm23 = 0.f;
    if (CT && (mode & MESH_GREEN)) {
        const int c = tid & (TW - 1);
        bm23 = b2[!RAG || c < W ? g20 + c : g20] * b3[m3];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int t = tid + u * NT;
            bm1[u] = (t < K1 * TW) ? b1[t >> twl] : 0.f;
        }
    }
    auto ld_tw = [&](int t) { return ax1.tw[t]; };
    auto st_tw = [&](int t, float2 v) { tw[t] = v; };
    auto ld = [&](int t) {
        const int c = t & (TW - 1), g1 = t >> twl;
        return (!RAG || c < W) && m2_kept(k, g20 + c) ? base[(size_t)g1 * K2 + c] : make_float2(0.f, 0.f);
    };
    auto st = [&](int t, float2 v) { buf[t] = v; };
    if constexpr (CT) {
        stage2_ct<KC, KC * TWC, NT, float2>(tid, ld_tw, st_tw, ld, st);
    } else {
        stage_rt<4, float2>(K1, tid, NT, ld_tw, st_tw);
        stage_rt<4, float2>(K1 * TW, tid, NT, ld, st);
    }
    __syncthreads();
    if (mode & MESH_FWD) {
        if constexpr (KC > 0 && TWC > 0)
            fft_ct<KC, TWC, TWC, NT, false>(buf, tw, tid);
        else
            fft_lds(buf, ax1, twl, tw, false, tid, NT);
    }
    if (mode & MESH_GREEN) {
        double e = 0.0;
        const float mult = (m3 == 0) ? 1.f : 2.f;
        if constexpr (CT) {
            // a thread's elements share m2 (its column) and m3 (the block's):
            // the quadratic form k^2 / (2 pi)^2 = M11 x1^2 + l1 x1 + q23 is two
            // FMAs per element, and the screened kernel uses the hardware
            // exponential and reciprocal (a few ulp, far below the FP32
            // spectrum's own rounding where G is not already negligible)
            const int cc = tid & (TW - 1);
            const int m2 = !RAG || cc < W ? g20 + cc : g20;
            const float x2 = (float)(m2 <= k.K2 / 2 ? m2 : m2 - k.K2), x3 = (float)m3;
            const float M11 = (float)k.M[0];
            const float l1 = 2.0f * ((float)k.M[3] * x2 + (float)k.M[4] * x3);
            const float q23 = (float)k.M[1] * x2 * x2 + (float)k.M[2] * x3 * x3 + 2.0f * (float)k.M[5] * x2 * x3;
            const float eta = (float)k.eta_green;
            // exp(-eta^2 k^2 / 2) = 2^(ce q): ce = -eta^2 (2 pi)^2 log2(e) / 2
            const float ce = -0.5f * eta * eta * 39.478417604357434475f * 1.4426950408889634f;
            const float pref = (float)k.green_pref / 39.478417604357434475f;
            const bool nyq23 = 2 * m2 == k.K2 || 2 * m3 == k.K3;
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const int t = tid + u * NT;
                if (t >= K1 * TW) break;
                const int m1 = t >> twl;
                const float x1 = (float)(m1 <= K1 / 2 ? m1 : m1 - K1);
                const float q = fmaf(fmaf(M11, x1, l1), x1, q23);
                float g = pref * __builtin_amdgcn_exp2f(ce * q) * __builtin_amdgcn_rcpf(q) * (bm1[u] * bm23);
                if (nyq23 || 2 * m1 == K1 || (m1 | m2 | m3) == 0) g = 0.f;
                const float2 x = buf[t];
                if (mode & MESH_ENERGY) e += (double)(g * mult * (x.x * x.x + x.y * x.y));
                buf[t] = make_float2(x.x * g, x.y * g);
            }
        } else {
            for (int t = tid; t < K1 * TW; t += NT) {
                const int c = t & (TW - 1), m1 = t >> twl;
                const float g = green_value(k, m1, g20 + c, m3, b1, b2, b3);
                const float2 x = buf[t];
                if (mode & MESH_ENERGY) e += (double)(g * mult * (x.x * x.x + x.y * x.y));
                buf[t] = make_float2(x.x * g, x.y * g);
            }
        }
        if (mode & MESH_ENERGY) {
            double v[1] = {e};
            block_sum<1>(v);
            if (tid == 0) epart[blockIdx.x] = v[0];
        }
        __syncthreads();
    }
    if (mode & MESH_INV) {
        if constexpr (KC > 0 && TWC > 0)
            fft_ct<KC, TWC, TWC, NT, true>(buf, tw, tid);
        else
            fft_lds(buf, ax1, twl, tw, true, tid, NT);
    }
    for (int t = tid; t < K1 * TW; t += NT) {
        const int c = t & (TW - 1), g1 = t >> twl;
        if ((!RAG || c < W) && m2_kept(k, g20 + c)) base[(size_t)g1 * K2 + c] = buf[t];
    }
}

// ------------------------------------------------------------------ pass 5
template <int KC, int TWC, bool RAG = false>
__global__ __launch_bounds__(NT) void k_c2r(KParams k, FftAxis ax3, const float2* __restrict__ C,
                                           float* __restrict__ R, const int* __restrict__ done) {
    if (done && *done) return;
    extern __shared__ float2 sm[];
    const int K3 = KC ? KC : k.K3;
    const int TW = TWC ? TWC : k.TW;
    const int K3h = K3 / 2 + 1;
    const int K1 = k.K1, K2 = k.K2;
    const int ncol = TW >> 1;
    const int twl = ilog2_dev(TW);
    const int ncl = twl - 1;
    float2* tw = sm;
    float2* X = sm + K3;
    float2* Z = X + K3h * TW;
    const int tid = threadIdx.x;
    const int g1 = blockIdx.x / k.ntile;
    int g20, W;
    tile_of<RAG>(blockIdx.x - g1 * k.ntile, k.ntile, K2, TW, g20, W);
    {
        auto ld_tw = [&](int t) { return ax3.tw[t]; };
        auto st_tw = [&](int t, float2 v) { tw[t] = v; };
        auto ld = [&](int t) {
            const int r = t & (TW - 1), m = t >> twl;
            return m < k.K3h && (!RAG || r < W) ? C[((size_t)m * K1 + g1) * K2 + g20 + r] : make_float2(0.f, 0.f);
        };
        auto st = [&](int t, float2 v) { X[t] = v; };
        if constexpr (KC > 0 && TWC > 0) {
            stage2_ct<KC, (KC / 2 + 1) * TWC, NT, float2>(tid, ld_tw, st_tw, ld, st);
        } else {
            stage_rt<4, float2>(K3, tid, NT, ld_tw, st_tw);
            stage_rt<4, float2>(K3h * TW, tid, NT, ld, st);
        }
    }
    __syncthreads();
    // Z = X_even + i X_odd over the full axis (Hermitian extension)
    for (int t = tid; t < K3 * ncol; t += NT) {
        const int pr = t & (ncol - 1), m = t >> ncl;
        float2 xa, xb;
        if (2 * m <= K3) {
            xa = X[m * TW + 2 * pr];
            xb = X[m * TW + 2 * pr + 1];
        } else {
            xa = X[(K3 - m) * TW + 2 * pr];
            xb = X[(K3 - m) * TW + 2 * pr + 1];
            xa.y = -xa.y;
            xb.y = -xb.y;
        }
        Z[t] = make_float2(xa.x - xb.y, xa.y + xb.x);
    }
    __syncthreads();
    if constexpr (KC > 0 && TWC > 0)
        fft_ct<KC, TWC / 2, TWC / 2, NT, true>(Z, tw, tid);
    else
        fft_lds(Z, ax3, ncl, tw, true, tid, NT);
    const float* zf = reinterpret_cast<const float*>(Z);
    for (int t = tid; t < W * K3; t += NT) {
        const int r = t / K3;
        const int g3 = t - r * K3;
        R[((size_t)g1 * K2 + g20 + r) * K3 + g3] = zf[(g3 * ncol + (r >> 1)) * 2 + (r & 1)];
    }
}

// ------------------------------------------------------------------ pass 5 fused with interpolation
// The complex-to-real pass of a (g1, TW-row) tile followed, while the tile's
// potential is still in LDS, by the part of every atom's back-interpolation
// (eq. matvec: the integral of the potential over the atom's charge
// distribution, here sum_g theta_i(g) phi(g)) that falls on this tile, so the
// real grid is never written or read again:
//   partial = w1(k1) sum_{k2: row in tile} w2(k2) sum_k3 w3(k3) phi(g1, h2 - k2, h3 - k3)
// for every atom with h1 = g1 + k1 (k1 < p) whose rows h2 - p + 1 .. h2 meet
// the tile (TW >= p - 1, so at most two tiles).  Each partial goes to its own
// slot, mpart[(2 k1 + t) n + atom] with t = 0 for the tile holding row h2 and
// t = 1 for the tile before it (written as 0 by the first when the atom's rows
// all lie in one tile): 2p FP32 partials per atom, summed in a fixed order by
// the pair-product kernel, so the result does not depend on block timing.
template <int KC, int TWC, int PC, bool RAG = false>
__global__ __launch_bounds__(NT) void k_c2r_interp(KParams k, FftAxis ax3, const float2* __restrict__ C,
                                                  const int* __restrict__ bin_start,
                                                  const int* __restrict__ home,
                                                  const float* __restrict__ wts, float* __restrict__ mpart,
                                                  const int* __restrict__ done) {
    if (done && *done) return;
    extern __shared__ float2 sm[];
    constexpr bool CT = KC > 0 && TWC > 0;
    const int K3 = KC ? KC : k.K3;
    const int TW = TWC ? TWC : k.TW;
    const int p = PC ? PC : k.p;
    const int K3h = K3 / 2 + 1;
    const int K1 = k.K1, K2 = k.K2;
    const int ncol = TW >> 1;
    const int twl = ilog2_dev(TW);
    const int ncl = twl - 1;
    float2* tw = sm;
    float2* X = sm + K3;
    // compile-time sizes: the packed rows Z (K3 x TW/2) replace X (K3/2 + 1
    // rows of TW) in place through registers, halving the block's LDS
    float2* Z = CT ? X : X + K3h * TW;
    __shared__ int seg_lo[2 * QEQ_MAXP], seg_len[2 * QEQ_MAXP], seg_off[2 * QEQ_MAXP + 1];
    const int tid = threadIdx.x;
    const int blk = xcd_remap(blockIdx.x, gridDim.x);
    const int g1 = blk / k.ntile;
    int g20, W;
    tile_of<RAG>(blk - g1 * k.ntile, k.ntile, K2, TW, g20, W);
    // candidate segments (as in the spread pass): homes h1 = g1 + k1,
    // h2 in [g20, g20 + TW + p - 1), two pieces when the range wraps
    if (tid < p) {
        const int k1 = tid;
        int h1 = g1 + k1;
        if (h1 >= K1) h1 -= K1;
        const int b0 = h1 * K2;
        const int hi = g20 + W + p - 1;
        const int e1 = hi < K2 ? hi : K2;
        const int lo0 = bin_start[b0 + g20];
        seg_lo[2 * k1] = lo0;
        seg_len[2 * k1] = bin_start[b0 + e1] - lo0;
        if (hi > K2) {
            const int lo1 = bin_start[b0];
            seg_lo[2 * k1 + 1] = lo1;
            seg_len[2 * k1 + 1] = bin_start[b0 + (hi - K2)] - lo1;
        } else {
            seg_lo[2 * k1 + 1] = 0;
            seg_len[2 * k1 + 1] = 0;
        }
    }
    {
        auto ld_tw = [&](int t) { return ax3.tw[t]; };
        auto st_tw = [&](int t, float2 v) { tw[t] = v; };
        auto ld = [&](int t) {
            const int r = t & (TW - 1), m = t >> twl;
            return m < k.K3h && (!RAG || r < W) ? C[((size_t)m * K1 + g1) * K2 + g20 + r] : make_float2(0.f, 0.f);
        };
        auto st = [&](int t, float2 v) { X[t] = v; };
        if constexpr (CT) {
            stage2_ct<KC, (KC / 2 + 1) * TWC, NT, float2>(tid, ld_tw, st_tw, ld, st);
        } else {
            stage_rt<4, float2>(K3, tid, NT, ld_tw, st_tw);
            stage_rt<4, float2>(K3h * TW, tid, NT, ld, st);
        }
    }
    __syncthreads();
    if (tid == 0) {
        int off = 0;
        for (int sg = 0; sg < 2 * p; ++sg) {
            seg_off[sg] = off;
            off += seg_len[sg];
        }
        seg_off[2 * p] = off;
    }
    // Z = X_even + i X_odd over the full axis (Hermitian extension)
    auto zval = [&](int t) {
        const int pr = t & (ncol - 1), m = t >> ncl;
        float2 xa, xb;
        if (2 * m <= K3) {
            xa = X[m * TW + 2 * pr];
            xb = X[m * TW + 2 * pr + 1];
        } else {
            xa = X[(K3 - m) * TW + 2 * pr];
            xb = X[(K3 - m) * TW + 2 * pr + 1];
            xa.y = -xa.y;
            xb.y = -xb.y;
        }
        return make_float2(xa.x - xb.y, xa.y + xb.x);
    };
    // compile-time sizes: the packed values are built inside the first radix
    // stage of the transform (each item reads the X elements of its R0 inputs
    // into registers; after the barrier the stage's outputs overwrite X in
    // place), so the packing costs no LDS pass of its own
    constexpr int NCZ = CT ? TWC / 2 : 1;
    constexpr int R0 = CT ? ct_radix_at(KC, 0, TWC / 2, NT) : 1;
    constexpr int PER0 = CT ? KC / R0 : 1;
    constexpr int IT0 = CT ? (PER0 * NCZ + NT - 1) / NT : 1;
    float2 v0[IT0][R0];
    if constexpr (CT) {
#pragma unroll
        for (int it = 0; it < IT0; ++it) {
            const int item = tid + it * NT;
            if ((PER0 * NCZ) % NT == 0 || item < PER0 * NCZ) {
                const int c = item % NCZ, j = item / NCZ;
#pragma unroll
                for (int r = 0; r < R0; ++r) v0[it][r] = zval((j + r * PER0) * NCZ + c);
            }
        }
    } else {
        for (int t = tid; t < K3 * ncol; t += NT) Z[t] = zval(t);
    }
    __syncthreads();
    // the first round's candidate is fetched before the transform so that its
    // loads overlap it
    const int ncand = seg_off[2 * p];
    const int n = k.n;
    constexpr int PM = PC ? PC : QEQ_MAXP;
    float w1 = 0.f, w2[PM], w3[PM];
    int a = 0, k1 = 0, h2 = 0, h3 = 0;
    auto load_cand = [&](int cidx) {
        // last segment starting at or before cidx (empty segments are passed over)
        int sg = 0;
#pragma unroll
        for (int s2 = 1; s2 < 2 * PM; ++s2) {
            if (!PC && s2 >= 2 * p) break;
            sg += cidx >= seg_off[s2] ? 1 : 0;
        }
        k1 = sg >> 1;
        a = seg_lo[sg] + (cidx - seg_off[sg]);
        const float* w = wts + (size_t)a * 3 * QEQ_MAXP;
        w1 = w[k1];
#pragma unroll
        for (int kk = 0; kk < PM; ++kk) {
            if (!PC && kk >= p) break;
            w2[kk] = w[QEQ_MAXP + kk];
            w3[kk] = w[2 * QEQ_MAXP + kk];
        }
        h2 = home[4 * a + 1];
        h3 = home[4 * a + 2];
    };
    if (tid < ncand) load_cand(tid);
    if constexpr (CT) {
#pragma unroll
        for (int it = 0; it < IT0; ++it) {
            const int item = tid + it * NT;
            if ((PER0 * NCZ) % NT == 0 || item < PER0 * NCZ) {
                const int c = item % NCZ, j = item / NCZ;
                dft<R0>(v0[it], true);
#pragma unroll
                for (int r = 0; r < R0; ++r) Z[(j * R0 + r) * NCZ + c] = v0[it][r];
            }
        }
        __syncthreads();
        fft_ct<KC, TWC / 2, TWC / 2, NT, true, 1, R0>(Z, tw, tid);
    } else {
        fft_lds(Z, ax3, ncl, tw, true, tid, NT);
    }
    // phi(g1, g20 + r, g3) = zf[(g3 ncol + r / 2) 2 + r % 2]
    const float* zf = reinterpret_cast<const float*>(Z);
    for (int cidx = tid; cidx < ncand; cidx += NT) {
        if (cidx != tid) load_cand(cidx);
        int d = h2 - g20;
        if (d < 0) d += K2;
        float s = 0.f;
#pragma unroll
        for (int k2 = 0; k2 < PM; ++k2) {
            if (!PC && k2 >= p) break;
            const int r = d - k2;
            if (r < 0 || r >= W) continue;
            const float* zr = zf + (r >> 1) * 2 + (r & 1);
            float t = 0.f;
#pragma unroll
            for (int k3 = 0; k3 < PM; ++k3) {
                if (!PC && k3 >= p) break;
                int g3 = h3 - k3;
                if (g3 < 0) g3 += K3;
                t += w3[k3] * zr[g3 * ncol * 2];
            }
            s += w2[k2] * t;
        }
        const int slot = 2 * k1 + (d < W ? 0 : 1);
        mpart[(size_t)slot * n + a] = w1 * s;
        if (d < W && d >= p - 1) mpart[(size_t)(slot + 1) * n + a] = 0.f;
    }
}

// Strain factor of one mode: under r -> (1 + eps) r (fractional coordinates
// fixed) k -> (1 + eps)^-T k and V -> (1 + tr eps) V, so
//   d ln G(m) / d eps_ab = -delta_ab + 2 (1/k^2 + eta^2/2) k_a k_b
// (the B-spline moduli do not change).  kv = 2 pi H^-1 m, returns k^2.
__device__ __forceinline__ float mode_kvec(const KParams& k, int m1, int m2, int m3, float kv[3]) {
    const float x1 = (float)(m1 <= k.K1 / 2 ? m1 : m1 - k.K1);
    const float x2 = (float)(m2 <= k.K2 / 2 ? m2 : m2 - k.K2);
    const float x3 = (float)m3;
    float k2 = 0.f;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        kv[c] = 6.283185307179586477f * ((float)k.Hinv[c * 3] * x1 + (float)k.Hinv[c * 3 + 1] * x2 +
                                         (float)k.Hinv[c * 3 + 2] * x3);
        k2 += kv[c] * kv[c];
    }
    return k2;
}

// Virial of the reciprocal mesh energy E = 1/2 sum_m G(m) |Q(m)|^2: the
// axis-1 forward transform of a column tile (the grid already transformed
// along axes 3 and 2), then per mode e = G |Q|^2 (doubled off the m3 = 0
// plane) and per block the sums of e and of e c k_a k_b, c = 2 (1/k^2 + eta^2/2);
// W = 1/2 (sum e) delta - 1/2 sum e c k k.  The grid is left as it is.
template <int KC, int TWC, bool RAG = false>
__global__ __launch_bounds__(NT) void k_cols_virial(KParams k, FftAxis ax1, const float2* __restrict__ C,
                                                   const float* __restrict__ b1, const float* __restrict__ b2,
                                                   const float* __restrict__ b3, double* __restrict__ part) {
    extern __shared__ float2 sm[];
    const int K1 = KC ? KC : k.K1;
    const int TW = TWC ? TWC : k.TW;
    const int twl = ilog2_dev(TW);
    float2* tw = sm;
    float2* buf = sm + K1;
    const int tid = threadIdx.x;
    const int K2 = k.K2;
    const int m3 = blockIdx.x / k.ntile;
    int g20, W;
    tile_of<RAG>(blockIdx.x - m3 * k.ntile, k.ntile, K2, TW, g20, W);
    for (int t = tid; t < K1; t += NT) tw[t] = ax1.tw[t];
    const float2* base = C + (size_t)m3 * K1 * K2 + g20;
    for (int t = tid; t < K1 * TW; t += NT) {
        const int c = t & (TW - 1), g1 = t >> twl;
        buf[t] = (!RAG || c < W) && m2_kept(k, g20 + c) ? base[(size_t)g1 * K2 + c] : make_float2(0.f, 0.f);
    }
    __syncthreads();
    if constexpr (KC > 0 && TWC > 0)
        fft_ct<KC, TWC, TWC, NT, false>(buf, tw, tid);
    else
        fft_lds(buf, ax1, twl, tw, false, tid, NT);
    double v[7] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    const float mult = (m3 == 0) ? 1.f : 2.f;
    const float eta = (float)k.eta;
    for (int t = tid; t < K1 * TW; t += NT) {
        const int c = t & (TW - 1), m1 = t >> twl;
        if ((RAG && c >= W) || !m2_kept(k, g20 + c)) continue;
        const float g = green_value(k, m1, g20 + c, m3, b1, b2, b3);
        if (g == 0.f) continue;
        const float2 x = buf[t];
        float kv[3];
        const float k2 = mode_kvec(k, m1, g20 + c, m3, kv);
        const float e = g * mult * (x.x * x.x + x.y * x.y);
        const float ec = e * 2.f * (1.f / k2 + 0.5f * eta * eta);
        v[0] += (double)e;
        v[1] += (double)(ec * kv[0] * kv[0]);
        v[2] += (double)(ec * kv[1] * kv[1]);
        v[3] += (double)(ec * kv[2] * kv[2]);
        v[4] += (double)(ec * kv[0] * kv[1]);
        v[5] += (double)(ec * kv[0] * kv[2]);
        v[6] += (double)(ec * kv[1] * kv[2]);
    }
    block_sum<7>(v);
    if (tid == 0)
        for (int u = 0; u < 7; ++u) part[(size_t)blockIdx.x * QEQ_NPART + u] = v[u];
}

}  // namespace
