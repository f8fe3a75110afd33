// The words that windows of the bf16 / d = 128 compression tell each other their rows with.  Every word can be read without any other: a reader
// combines words that were read at different moments.
#pragma once
#include <stdint.h>

namespace sc {

// A window's word: kPubRows and the rows, as soon as they are known; kPubReady: a long chunk, and the clusters of its rows have arrived;
// kPubLeft: its workgroup has stopped waiting and has left the merged rows to others.
constexpr uint32_t kPubRows = 1u << 30, kPubReady = 1u << 31, kPubLeft = 1u << 29;
constexpr uint32_t kPubValue = (1u << 29) - 1u;

// A segment's words.  `part`: in the low bits, as many as segment_bits says, the windows that have not published yet; above them the rows of
// those that have.  `upto`: kPubRows and the rows of the sequence up to the segment's end, once somebody has found them.
struct GscSegment {
    uint32_t part, upto;
};
constexpr int segment_bits(int slots) {       // for 0 .. slots windows
    int bits = 1;
    while ((1 << bits) <= slots) ++bits;
    return bits;
}
constexpr bool segment_holds(int slots, int64_t rows) { return rows <= (int64_t)kPubValue && rows < (int64_t(1) << (32 - segment_bits(slots))); }
constexpr uint32_t segment_start(int windows) { return (uint32_t)windows; }
constexpr uint32_t segment_added(int rows, int bits) { return ((uint32_t)rows << bits) - 1u; }      // what a window adds to `part`
// rows of a segment's windows, if all are there
constexpr bool segment_complete(uint32_t part, int bits) { return (part & ((1u << bits) - 1u)) == 0u; }
constexpr int segment_rows(uint32_t part, int bits) { return (int)(part >> bits); }

// A (sequence, head)'s word: kHeadLeft: windows have been left; kHeadFailed: rows that had been published did not arrive.
constexpr uint32_t kHeadLeft = 1u, kHeadFailed = 2u;

}  // namespace sc
