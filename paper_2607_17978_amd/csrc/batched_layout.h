// Memory layout of the batched solve (batched.hip).  Plain C++, so that host
// tests compile it as it is; constexpr functions also run on the device.
#pragma once

#include <stddef.h>

namespace qeqb {

constexpr int BQ_KAX = 64;      // longest grid axis of a batched structure
constexpr int BQ_MAXP = 8;      // highest spline order
constexpr int BQ_NV = 11;       // per-atom FP64 vectors in a slot

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
