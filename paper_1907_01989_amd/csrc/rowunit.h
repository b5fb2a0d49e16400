// Index arithmetic of the input band's unaligned copy, apart from the kernels
// so that host code can check it too (a constexpr function is callable on both
// sides).
#pragma once

namespace mgi {
namespace kern {

// Row floor(e / rowlen) of value e of a stretch of rows of rowlen >= 1 values,
// for e >= -vec: the first unit of vec values may start before the stretch, by
// more than a row where rows are shorter than a unit, so vec rows are added
// before the division, which keeps the dividend non-negative.
constexpr int unit_row(int e, int rowlen, int vec) {
    return (int)((unsigned)(e + vec * rowlen) / (unsigned)rowlen) - vec;
}

}  // namespace kern
}  // namespace mgi
