// The launches of one group of axis lengths (see mesh_len.h).
#pragma once

#include "mesh_len.h"
#include "mesh_passes.h"

namespace {

template <typename F>
int len_smem(F fn, size_t sh) {
    if (sh <= 65536) return QEQ_OK;   // the default window
    return qeq_check(hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh));
}

#define LEN_GO(FN, GRID, SH, ...)                                                                        \
    do {                                                                                                 \
        QEQ_TRY(len_smem(FN, SH));                                                                       \
        hipExtLaunchKernelGGL(FN, dim3((unsigned)(GRID)), dim3(NT), SH, pl->stream, c.ev0, c.ev1, 0, k,   \
                              __VA_ARGS__);                                                              \
        return qeq_check(hipGetLastError());                                                             \
    } while (0)

template <int KC>
int len_launch(const LenCall& c) {
    qeq_plan* pl = c.pl;
    const KParams& k = pl->kp;
    constexpr int TW = LEN_TW, NR = len_nr(KC);
    constexpr size_t cx = sizeof(float2);
    const size_t sh_half = cx * (KC + (size_t)(KC / 2 + 1) * TW);
    switch (c.pass) {
        case LEN_SPREAD: {
            const size_t sh = cx * KC + sizeof(int) * (size_t)KC * TW;
            if (k.p == 6)
                LEN_GO((k_spread_r2c<KC, TW, 6, true>), k.K1 * k.ntile_s, sh, pl->axes.ax[2], c.src, pl->bin_start,
                       pl->home, pl->wts, pl->grid_c, c.done);
            LEN_GO((k_spread_r2c<KC, TW, 0, true>), k.K1 * k.ntile_s, sh, pl->axes.ax[2], c.src, pl->bin_start,
                   pl->home, pl->wts, pl->grid_c, c.done);
        }
        case LEN_ROWS_FWD:
        case LEN_ROWS_INV: {
            const int nrows = k.K3h * k.K1;
            const size_t sh = cx * (KC + (size_t)KC * (NR + 1));
            if (c.pass == LEN_ROWS_INV)
                LEN_GO((k_fft_rows<KC, NR, true>), (nrows + NR - 1) / NR, sh, pl->axes.ax[1], pl->grid_c, nrows,
                       c.done);
            LEN_GO((k_fft_rows<KC, NR, false>), (nrows + NR - 1) / NR, sh, pl->axes.ax[1], pl->grid_c, nrows, c.done);
        }
        case LEN_COLS:
            LEN_GO((k_fft_cols<KC, TW, true>), k.K3h * k.ntile, cx * (KC + (size_t)KC * TW), pl->axes.ax[0],
                   pl->grid_c, c.b1, c.b2, c.b3, c.mode, c.part, c.done);
        case LEN_VIRIAL:
            LEN_GO((k_cols_virial<KC, TW, true>), k.K3h * k.ntile, cx * (KC + (size_t)KC * TW), pl->axes.ax[0],
                   pl->grid_c, pl->bmod[0], pl->bmod[1], pl->bmod[2], c.part);
        case LEN_C2R:
            LEN_GO((k_c2r<KC, TW, true>), k.K1 * k.ntile, sh_half + cx * (size_t)KC * (TW / 2), pl->axes.ax[2],
                   pl->grid_c, pl->grid_r, c.done);
        case LEN_R2C:
            LEN_GO((k_r2c<KC, TW>), k.K1 * k.ntile, cx * (KC + (size_t)KC * (TW / 2)), pl->axes.ax[2], pl->grid_r,
                   pl->grid_c, c.done);
        case LEN_C2R_INTERP:
            if (k.p == 6)
                LEN_GO((k_c2r_interp<KC, TW, 6, true>), k.K1 * k.ntile, sh_half, pl->axes.ax[2], pl->grid_c,
                       pl->bin_start, pl->home, pl->wts, pl->mpart, c.done);
            LEN_GO((k_c2r_interp<KC, TW, 0, true>), k.K1 * k.ntile, sh_half, pl->axes.ax[2], pl->grid_c,
                   pl->bin_start, pl->home, pl->wts, pl->mpart, c.done);
    }
    return QEQ_EPLAN;
}

#undef LEN_GO

}  // namespace

#define QEQ_LEN_CASE(KK) case KK: return len_launch<KK>(c);
#define QEQ_LEN_GROUP(NAME, LIST)           \
    int NAME(const LenCall& c, int K) {     \
        switch (K) {                        \
            LIST(QEQ_LEN_CASE)              \
            default: return 1;              \
        }                                   \
    }
