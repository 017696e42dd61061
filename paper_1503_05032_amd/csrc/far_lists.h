// The whole numbers behind the lists of k_far_gather, which the kernels and the host form alike.
#ifndef CSR5_FAR_LISTS_H
#define CSR5_FAR_LISTS_H

#include <cstdint>

// Entries of a workgroup, workgroups of a segment, what a block's list in a chunk is padded to, blocks of x, the buffer.
constexpr int FAR_ENTRIES = 8192, FAR_SEGMENT = 64, FAR_PAD = 16, FAR_BLOCK_BYTES = 128 << 10, FAR_MAX_BLOCKS = 1024;
constexpr int64_t FAR_BUFFER_BYTES = 256 << 20;

// How many chunks `total` far entries go through the buffer in, and behind how many of them chunk c begins: with the
// first segment that has as many before it.  By the counted entries, since these may lie in any part of the rows. A chunk has one segment
// more than its even share at most, and every block's padding: with that it still fits the buffer.
constexpr int far_chunks(uint32_t total, int value_bytes) {
    const int64_t room = FAR_BUFFER_BYTES / value_bytes - int64_t(FAR_SEGMENT) * FAR_ENTRIES - FAR_MAX_BLOCKS * (FAR_PAD - 1) - 1;
    return int(total / room) + 1;
}
constexpr int FAR_MAX_CHUNKS = far_chunks(0x7fffffffu, 8);
constexpr uint32_t far_chunk_target(uint32_t total, int chunks, int chunk) { return uint32_t(uint64_t(total) * uint32_t(chunk) / uint32_t(chunks)); }

// The segment that chunk c begins with, from the workgroups' places in the list of all far entries (base[groups]: total)
constexpr int far_chunk_segment(const uint32_t* base, int segments, uint32_t total, int chunks, int chunk) {
    if (chunk == 0 || chunk == chunks) return chunk ? segments : 0;
    const uint32_t target = far_chunk_target(total, chunks, chunk);
    int lo = 0, hi = segments;
    while (lo < hi) {
        const int mid = (lo + hi) / 2;
        if (base[int64_t(mid) * FAR_SEGMENT] < target) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// A workgroup's share of a block's list [lo, hi), where `pieces` of them share it
struct FarPiece {
    uint32_t begin, end;
    constexpr FarPiece(uint32_t lo, uint32_t hi, int piece, int pieces) : begin(0), end(0) {
        const uint32_t share = ((hi - lo) / uint32_t(pieces) + FAR_PAD) / FAR_PAD * FAR_PAD;
        begin = lo + share * uint32_t(piece);
        end = begin + share < hi ? begin + share : hi;
    }
    constexpr bool empty() const { return begin >= end; }
};

#endif  // CSR5_FAR_LISTS_H
