// Sizes and index rules of the batched solve (batched.hip).  Plain C++, so that host
// tests compile it as it is; constexpr functions also run on the device.
#pragma once

#include <stddef.h>

namespace qeqb {

constexpr int BQ_KAX = 64;      // longest grid axis of a batched structure
constexpr int BQ_MAXP = 8;      // highest spline order
constexpr int BQ_NV = 11;       // per-atom FP64 vectors in a slot
constexpr int BQ_NC = 64;       // complex lines of a block along axis 3 (two real rows each) and axis 1
constexpr int BQ_KS = 65;       // their LDS row stride
constexpr int BQ_NC2 = 56;      // half-spectrum columns of a block along axis 2
constexpr int BQ_KS2 = 57;      // their LDS row stride
constexpr int BQ_NT = 512;      // threads of the plane and line kernels
constexpr int BQ_PB = 8;        // most planes of a block
constexpr size_t BQ_ACC = 38400;   // most bytes of a block's accumulator

constexpr int bq_min(int a, int b) { return a < b ? a : b; }
constexpr size_t bq_max(size_t a, size_t b) { return a > b ? a : b; }

// Planes of a block of k_bq_inv (km kept m3, spline order p) and of k_bq_fwd.
constexpr int bq_planes_inv(int K1, int K2, int km, int p) {
    const int n = bq_min(bq_min(2 * BQ_NC / K2, BQ_NC2 / km), bq_min(K1 - p + 1, BQ_PB));
    return n > 1 ? n : 1;
}
constexpr int bq_planes_fwd(int pb, int K2, int K3) {
    const int n = bq_min(pb, (int)(BQ_ACC / (8 * (size_t)K2 * K3)));
    return n > 1 ? n : 1;
}

// Bytes of LDS: lines along axis 1; lines along axis 3 and columns along axis 2
// in one place; the same with the accumulator of pf planes.
constexpr size_t bq_lds_lines(int K1) { return 8 * (size_t)K1 * BQ_KS; }
constexpr size_t bq_lds_inv(int K2, int K3) { return bq_max(8 * (size_t)K3 * BQ_KS, 8 * (size_t)K2 * BQ_KS2); }
constexpr size_t bq_lds_fwd(int K2, int K3, int pf) { return bq_max(bq_lds_inv(K2, K3), 8 * (size_t)K3 * pf * K2); }

// Axis-2 index of the kept row e of a plane of the half spectrum, nm2 of K2 kept.
constexpr int bq_m2(int e, int nm2, int K2) { return e < ((nm2 + 1) >> 1) ? e : e + (K2 - nm2); }

// A thread's elements of a block's half spectra C[j nm2 + e][m]: 32 lanes along
// m (at most two steps: km <= 33), BQ_NT / 32 rows at a time, so that a step
// costs a carry instead of two divisions.  at: the row's place in X2[m2][j km].
struct BqWalk {
    static constexpr int ROWS = BQ_NT / 32;
    int nm2, km, half, skip, j, e, row;
    constexpr BqWalk(int tid, int nm2_, int km_, int K2)
        : nm2(nm2_), km(km_), half((nm2_ + 1) >> 1), skip(K2 - nm2_), j(0), e(tid >> 5), row(tid >> 5) {
        carry();
    }
    constexpr void carry() {
        while (e >= nm2) {
            e -= nm2;
            ++j;
        }
    }
    constexpr int at() const { return (e < half ? e : e + skip) * BQ_KS2 + j * km; }
    constexpr void next() {
        row += ROWS;
        e += ROWS;
        carry();
    }
};

// Offsets inside one structure's scratch slot, in units of 256 bytes: 1,024
// atoms with a cutoff of four cell widths have 2.8e8 pairs of 24 bytes, past 32
// bits of bytes.  64-bit byte offsets cost every kernel of a product twice the
// scalar registers for them (1,024 structures 18.26 -> 18.42 ms).
struct BSlot {
    unsigned C, G, wts, dwts, home, frac, vec, selfgrad, row, col, kval, pdr, tab, mpart, hstart, perm, fpair;
};

constexpr size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
constexpr size_t slot_bytes(unsigned units) { return (size_t)units << 8; }

// Offsets of the slot of n atoms, nhalf kept half-spectrum points and room for
// pcap pairs; returns its size.
constexpr size_t slot_layout(BSlot& L, size_t n, size_t nhalf, size_t pcap) {
    constexpr size_t f32 = 4, f64 = 8, i32 = 4, np = 2 * BQ_MAXP - 1;
    size_t o = 0;
    auto place = [&o](size_t bytes) {
        const unsigned at = (unsigned)(o >> 8);
        o = align256(o + bytes);
        return at;
    };
    L.C = place(2 * f32 * nhalf);
    L.G = place(f32 * nhalf);
    L.wts = place(f32 * 3 * BQ_MAXP * n);
    L.dwts = place(f32 * 3 * BQ_MAXP * n);
    L.home = place(i32 * 4 * n);
    L.frac = place(f64 * 3 * n);
    L.vec = place(f64 * BQ_NV * n);
    L.selfgrad = place(f64 * 3 * n);
    L.row = place(2 * i32 * n);
    L.col = place(i32 * pcap);
    L.kval = place(f32 * pcap);
    L.pdr = place(4 * f32 * pcap);
    L.tab = place(f64 * np * np * np);
    L.mpart = place(f32 * 4 * BQ_MAXP * n);
    L.hstart = place(i32 * (BQ_KAX + 1));
    L.perm = place(i32 * n);
    L.fpair = place(f64 * 3 * n);
    return o;
}

}  // namespace qeqb
