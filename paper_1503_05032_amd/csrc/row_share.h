// The rows that one thread of a workgroup looks after where all m rows of a matrix are shared
// out evenly among `groups` workgroups, and a workgroup's rows are taken by its threads in turn.
#ifndef CSR5_ROW_SHARE_H
#define CSR5_ROW_SHARE_H

#include <cstdint>

// Unsigned: m may be 2^31 - 2, and the step behind a last row has to stay representable.
struct RowShare {
    uint32_t row, end;
    constexpr RowShare(int32_t m, uint32_t group, uint32_t groups, uint32_t thread)
        : row(uint32_t(uint64_t(m) * group / groups) + thread), end(uint32_t(uint64_t(m) * (group + 1) / groups)) {}
    constexpr bool more() const { return row < end; }
    constexpr void next(uint32_t threads) { row += threads; }
};

#endif  // CSR5_ROW_SHARE_H
