// Compile-time mesh passes for every supported axis length (multiples of 4
// with prime factors 2, 3, 5, from 12 to 512): one translation unit per group
// of lengths (mesh_len_*.hip), so that they compile side by side.
#pragma once

#include "internal.h"

enum LenPass { LEN_SPREAD, LEN_ROWS_FWD, LEN_ROWS_INV, LEN_COLS, LEN_VIRIAL, LEN_C2R, LEN_C2R_INTERP, LEN_R2C };

struct LenCall {
    qeq_plan* pl;
    LenPass pass;
    const double* src;       // LEN_SPREAD: charges
    int mode;                // LEN_COLS: MESH_* bits
    double* part;            // LEN_COLS: energy partials; LEN_VIRIAL: partial sums
    const float *b1, *b2, *b3;   // LEN_COLS: moduli
    const int* done;
    hipEvent_t ev0, ev1;
};

// Row tiles of the ragged passes: as many of at most LEN_TW rows as it takes,
// at least two (with one, an atom's rows would wrap into the tile they left).
constexpr int LEN_TW = 16;
inline int len_tiles(int K2) { return K2 <= 2 * LEN_TW ? 2 : (K2 + LEN_TW - 1) / LEN_TW; }
inline int len_rows_min(int K2) { return 2 * ((K2 / 2) / len_tiles(K2)); }
inline int len_rows_max(int K2) { return 2 * ((K2 / 2 + len_tiles(K2) - 1) / len_tiles(K2)); }

// Rows per block of the axis-2 pass: 16 within 32 KB of LDS; from 300 on, where
// a cubic grid streams from HBM, four (as for the 320 rows of mesh.hip: 58 ->
// 53 us forward, 54 -> 46 us inverse against eight).
constexpr int len_nr(int K2) { return K2 >= 300 ? 4 : (K2 > 256 ? 8 : 16); }

// Launches the pass for axis length K; 1 if the group does not hold K.
int mesh_len_a(const LenCall& c, int K);
int mesh_len_b(const LenCall& c, int K);
int mesh_len_c(const LenCall& c, int K);
int mesh_len_d(const LenCall& c, int K);
int mesh_len_e(const LenCall& c, int K);
int mesh_len_f(const LenCall& c, int K);
int mesh_len_g(const LenCall& c, int K);
int mesh_len_h(const LenCall& c, int K);

inline int mesh_len(const LenCall& c, int K) {
    int (*const groups[])(const LenCall&, int) = {mesh_len_a, mesh_len_b, mesh_len_c, mesh_len_d,
                                                  mesh_len_e, mesh_len_f, mesh_len_g, mesh_len_h};
    for (auto g : groups) {
        const int rc = g(c, K);
        if (rc != 1) return rc;
    }
    return QEQ_EPLAN;
}
