// How a walk workgroup cuts the bounding box of its batch's cells into pieces
// whose windows of the activity field fit in LDS.  Plain C++ for host and
// device (constexpr functions are both).
#pragma once

#include <cstdint>

namespace vr {

// A window of the activity field staged in LDS: up to kWalkSide x kWalkSide
// cells in rows of kWalkPitch words (odd, so that a column spreads over the
// LDS banks).
constexpr int32_t kWalkSide = 64, kWalkPitch = 65;

struct WalkPieces {
    uint32_t split;   // pieces a side
    bool windowed;    // their windows are staged
};

// A box of bw x bh cells, moves of at most `longest` cells: as few pieces as
// let each one, grown by the longest move, fit a window, and as many as there
// are workgroups (`parts`).  A piece costs a few barriers and a window whatever
// its cells: short searches over many pieces are quicker from memory (49 moves,
// 100,000 agents on 200 x 200 cells: 31.7 us in pieces, 17.8 us without), so a
// piece has to save the search of 16 moves.
constexpr WalkPieces walk_pieces(uint32_t bw, uint32_t bh, uint32_t longest, uint32_t parts, uint32_t num_moves) {
    const uint32_t least = parts >= 16 ? 4u : parts >= 4 ? 2u : 1u;
    if (2 * longest >= (uint32_t)kWalkSide) return {least, false};
    const uint32_t room = (uint32_t)kWalkSide - 2 * longest;   // cells a side besides the margins
    // ceil(box / split) <= room exactly when split >= ceil(box / room)
    const uint32_t box = bw > bh ? bw : bh, need = (box + room - 1) / room;
    const uint32_t split = need > least ? need : least;
    // at most 65,535 moves: none allows 65 pieces a side, and the product stays small
    return {split, split <= 64 && 16 * split * split <= num_moves};
}

}  // namespace vr
