// The middle of the particle-mesh product in one pass, for grids whose m3
// planes fit the LDS of one CU: per kept m3 plane the forward axis-2 and
// axis-1 transforms, the Green's function, and both inverse transforms, in
// place of three passes over the half spectrum (rows, columns, rows).
//
// Small grids are bound by launches and barriers, not by bytes: a pass costs 3
// to 4 us whatever it moves, and its successor's loads another microsecond.
// One block per plane leaves most CUs idle, so the work of a plane has to stay
// small.  Against the three passes, us a product: 24^3 10.1 -> 6.2, 48^3 12.4
// -> 9.4, 40 x 60 x 60 13.2 -> 10.2; beyond 64 it loses (80^3 13 -> 19, 128^3 17
// -> 29 in a build with longer lengths).  A solve of 64 atoms 600 -> 550 us, 512
// 860 -> 816, 1,000 1,085 -> 1,035; two steps of a 500-atom cell 3.64 -> 3.22 ms.
// Tiles of 32, 48 and 64 lines (lines a plane does not have are worked out and
// dropped: 48^3 10.2 us in tiles of 64), eight threads a line.
#include "internal.h"

namespace {

// Every supported axis length up to NCB: multiples of 4 with prime factors
// 2, 3, 5.
#define MID_LEN_32(X) X(12) X(16) X(20) X(24) X(32)
#define MID_LEN_48(X) X(36) X(40) X(48)
#define MID_LEN_64(X) X(60) X(64)

constexpr int mid_threads(int ncb) { return 8 * ncb; }

// Transform of length K over NCB lines: element i of line c at i * ES + c * CS.
template <int NCB, bool INV, int ES, int CS>
__device__ __forceinline__ void mid_fft(float2* buf, int K, const float2* tw, int tid) {
    constexpr int NT = mid_threads(NCB);
#define X(KK) case KK: fft_ct<KK, NCB, ES, NT, INV, 0, 1, CS>(buf, tw, tid); break;
    if (K <= 32) {
        switch (K) { MID_LEN_32(X) }
    }
    if constexpr (NCB >= 48) {
        switch (K) { MID_LEN_48(X) }
    }
    if constexpr (NCB >= 64) {
        switch (K) { MID_LEN_64(X) }
    }
#undef X
}

// One block per m3 plane; lines beyond K1 or K2 hold whatever the LDS held and
// are never stored.
template <int NCB>
__global__ __launch_bounds__(mid_threads(NCB)) void k_mid(KParams k, FftAxis ax1, FftAxis ax2,
                                                          float2* __restrict__ C, const float* __restrict__ b1,
                                                          const float* __restrict__ b2,
                                                          const float* __restrict__ b3,
                                                          const int* __restrict__ done) {
    if (done && *done) return;
    constexpr int NT = mid_threads(NCB), KS = NCB + 1, RPS = NT / NCB;   // rows a step
    constexpr int U = NCB / RPS;                                         // rows a thread
    extern __shared__ float2 sm[];
    float2* tw1 = sm;
    float2* tw2 = tw1 + NCB;
    float2* X = tw2 + NCB;   // [g1][g2], row stride KS
    const int tid = threadIdx.x, m3 = blockIdx.x;
    const int K1 = k.K1, K2 = k.K2;
    const int c = tid % NCB, r0 = tid / NCB;
    float2* base = C + (size_t)m3 * K1 * K2;
    float2 w = make_float2(0.f, 0.f);
    if (tid < K1) w = ax1.tw[tid];
    else if (tid >= NCB && tid - NCB < K2) w = ax2.tw[tid - NCB];
    const bool in2 = c < K2;
    const float b23 = in2 ? b2[c] * b3[m3] : 0.f;
    float2 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
        v[u] = in2 && r0 + u * RPS < K1 ? base[(size_t)(r0 + u * RPS) * K2 + c] : make_float2(0.f, 0.f);
#pragma unroll
    for (int u = 0; u < U; ++u) X[(r0 + u * RPS) * KS + c] = v[u];
    if (tid < 2 * NCB) tw1[tid] = w;   // tw1 and tw2 are contiguous
    __syncthreads();
    mid_fft<NCB, false, 1, KS>(X, K2, tw2, tid);
    mid_fft<NCB, false, KS, 1>(X, K1, tw1, tid);
    {
        // as the compile-time axis-1 pass: two FMAs a mode for k^2 / (2 pi)^2
        const float x2 = (float)(c <= K2 / 2 ? c : c - K2), x3 = (float)m3;
        const float M11 = (float)k.M[0];
        const float l1 = 2.0f * ((float)k.M[3] * x2 + (float)k.M[4] * x3);
        const float q23 = (float)k.M[1] * x2 * x2 + (float)k.M[2] * x3 * x3 + 2.0f * (float)k.M[5] * x2 * x3;
        const float eta = (float)k.eta_green;
        const float ce = -0.5f * eta * eta * 39.478417604357434475f * 1.4426950408889634f;
        const float pref = (float)k.green_pref / 39.478417604357434475f;
        const bool zero = 2 * c == K2 || 2 * m3 == k.K3 || !in2 || !(c <= k.M2 || c >= K2 - k.M2);
#pragma unroll 4
        for (int m1 = r0; m1 < K1; m1 += RPS) {
            const float x1 = (float)(m1 <= K1 / 2 ? m1 : m1 - K1);
            const float q = fmaf(fmaf(M11, x1, l1), x1, q23);
            float g = pref * __builtin_amdgcn_exp2f(ce * q) * __builtin_amdgcn_rcpf(q) * (b1[m1] * b23);
            if (zero || 2 * m1 == K1 || (m1 | c | m3) == 0) g = 0.f;
            const float2 x = X[m1 * KS + c];
            X[m1 * KS + c] = make_float2(x.x * g, x.y * g);
        }
    }
    __syncthreads();
    mid_fft<NCB, true, KS, 1>(X, K1, tw1, tid);
    mid_fft<NCB, true, 1, KS>(X, K2, tw2, tid);
    if (in2)
        for (int g1 = r0; g1 < K1; g1 += RPS) base[(size_t)g1 * K2 + c] = X[g1 * KS + c];
}

template <int NCB>
int mid_launch(qeq_plan* pl, const float* b1, const float* b2, const float* b3, const int* done, hipEvent_t e0,
               hipEvent_t e1) {
    const size_t sh = sizeof(float2) * ((size_t)2 * NCB + (size_t)NCB * (NCB + 1));
    hipExtLaunchKernelGGL((k_mid<NCB>), dim3(pl->kp.K3h), dim3(mid_threads(NCB)), sh, pl->stream, e0, e1, 0, pl->kp,
                          pl->axes.ax[0], pl->axes.ax[1], pl->grid_c, b1, b2, b3, done);
    return qeq_check(hipGetLastError());
}

}  // namespace

bool mid_available(const qeq_plan* pl) {
    const int K = pl->kp.K1 > pl->kp.K2 ? pl->kp.K1 : pl->kp.K2;
    return pl->fused_inverse && K <= MID_MAX;
}

int launch_mid(qeq_plan* pl, const float* b1, const float* b2, const float* b3, const int* done, hipEvent_t e0,
               hipEvent_t e1) {
    const int K = pl->kp.K1 > pl->kp.K2 ? pl->kp.K1 : pl->kp.K2;
    if (K <= 32) return mid_launch<32>(pl, b1, b2, b3, done, e0, e1);
    if (K <= 48) return mid_launch<48>(pl, b1, b2, b3, done, e0, e1);
    return K <= MID_MAX ? mid_launch<64>(pl, b1, b2, b3, done, e0, e1) : QEQ_EPLAN;
}
