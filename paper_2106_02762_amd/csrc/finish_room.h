// The scratch of the level peel's finish: the places of its arrays in one block of words, and how many
// (core, phase, degree class) cells a finish of R vertices counts.  Both stand here, beside the proof that no
// count of cells passes its array: the cells of R vertices grow with R (clearing them is part of a small
// finish's time) and end at the array's size.
#pragma once

#include <cstdint>

namespace dt {

constexpr uint32_t kTail = 65536;   // most vertices the finish takes (16-bit local ids and bounds)

struct FinishRoom {
    static constexpr uint32_t kCells = 1u << 18;   // (core, phase, class) cells counted in memory
    static constexpr uint32_t kClasses = 4;        // classes of degree over core number
    static constexpr uint64_t kBase = 0;                 // uint32[kCells]: first position of each cell
    static constexpr uint64_t kCur = kBase + kCells;     // uint32[kCells]: positions taken in each
    static constexpr uint64_t kWhen = kCur + kCells;     // uint32[kTail]: phase of each vertex
    static constexpr uint64_t kPos = kWhen + kTail;      // uint32[kTail]: its place in its cell
    static constexpr uint64_t kVal = kPos + kTail;       // uint16[2 * kTail]: two buffers of bounds
    static constexpr uint32_t kBlocks = 1024;            // blocks at most
    static constexpr uint64_t kFalls = kVal + kTail;     // uint32[2 * kBlocks]: two phases' falls, by block
    static constexpr uint64_t kWords = kFalls + 2 * kBlocks;
    // class of a vertex of core number k and degree d
    static constexpr uint32_t deg_class(uint32_t d, uint32_t k) {
        return d < 2 * k ? 0u : (d < 8 * k ? 1u : (d < 32 * k ? 2u : 3u));
    }
    // cells that a finish of R vertices uses at most
    static constexpr uint32_t cells(uint32_t R) {
        return R < (kCells - 1024) / 32 ? 32 * R + 1024 : kCells;
    }
};

constexpr bool finish_cells_fit() {
    for (uint32_t R = 1; R <= kTail; ++R)
        if (FinishRoom::cells(R) > FinishRoom::kCur - FinishRoom::kBase ||
            FinishRoom::cells(R) > FinishRoom::kWhen - FinishRoom::kCur || FinishRoom::cells(R) < R)
            return false;
    return true;
}
static_assert(finish_cells_fit(), "a finish's cells stay within their arrays");

}  // namespace dt
