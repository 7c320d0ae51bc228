// Do row-strided arrays of one common row stride share memory?  Host code.
#pragma once

#include <cstddef>
#include <cstdint>

namespace stk {

// The used extents of an array: `rows` rows of `width` bytes, `row` bytes apart.
struct Extent {
    const void* at;
    int64_t rows, width;
};

// Exact for extents of one row stride `row`, so that arrays laid out side by side in one
// allocation, whose rows interleave, do not count as shared.
inline bool share_memory(const Extent& a, const Extent& b, int64_t row) {
    // b's row 0 starts `row_off` rows and `col_off` bytes after a's
    const int64_t d = (int64_t)(reinterpret_cast<uintptr_t>(b.at) - reinterpret_cast<uintptr_t>(a.at));
    const int64_t row_off = d >= 0 ? d / row : -((-d + row - 1) / row), col_off = d - row_off * row;
    auto rows_meet = [&](int64_t off) { return off < a.rows && off > -b.rows; };
    return (col_off < a.width && rows_meet(row_off)) || (col_off + b.width > row && rows_meet(row_off + 1));
}

// Does a velocity pair share memory with a right-hand side of the same grid and layout?
// (es: bytes of an element; vx, bx: ny rows of nx + 1, vy, by: ny + 1 rows of nx)
inline bool velocity_shares(int nx, int ny, int64_t ld, int64_t es, const void* vx, const void* vy, const void* bx,
                            const void* by) {
    auto x = [&](const void* p) { return Extent{p, ny, ((int64_t)nx + 1) * es}; };
    auto y = [&](const void* p) { return Extent{p, (int64_t)ny + 1, nx * es}; };
    const int64_t row = ld * es;
    return share_memory(x(vx), x(bx), row) || share_memory(x(vx), y(by), row) || share_memory(y(vy), x(bx), row) ||
           share_memory(y(vy), y(by), row);
}

}  // namespace stk
