// Buffers that grow together and share one capacity.  Plain C++ with the
// allocator as a parameter, so that host tests can let it fail.
#pragma once

#include <stddef.h>

#include <initializer_list>

struct GrowBuf {
    void** p;
    size_t item;    // bytes per item
    size_t extra;   // items beyond the capacity
    bool fp;        // holds floating-point values
};

// Room for count items in every buffer (contents are not kept).  After a
// failed allocation none is left and cap is 0: a later request, however small,
// allocates again instead of taking a freed buffer for one of the old size.
template <typename Alloc, typename Free>
bool grow_together(size_t& cap, size_t count, std::initializer_list<GrowBuf> bufs, Alloc alloc, Free release) {
    if (count <= cap) return true;
    auto drop = [&]() {
        for (const GrowBuf& b : bufs) {
            if (*b.p) release(*b.p);
            *b.p = nullptr;
        }
    };
    cap = 0;
    drop();
    for (const GrowBuf& b : bufs) {
        *b.p = alloc(b, b.item * (count + b.extra));
        if (!*b.p) {
            drop();
            return false;
        }
    }
    cap = count;
    return true;
}
