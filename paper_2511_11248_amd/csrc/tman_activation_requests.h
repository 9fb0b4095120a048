// Which bytes a request for activations of the prefill kernel's pairs of stages touches.  Plain C++: the kernel
// and a test on the CPU use the same functions.
#pragma once
#include <cstdint>

namespace tman {

constexpr uint32_t kPairBytes = 128;  // of a token: two stages of 32 fp16 columns, a whole cache line

// Request q of a pair brings token rows 8 q .. 8 q + 7 straight into LDS, lane 8 R + P to place P of row 8 q + R.  16-byte chunk c
// of row R is kept at place c ^ ((R >> 1) & 7): the operand reads of 16 consecutive rows then fall into 16 different bank groups.
// The bytes of its row's 128 that a lane picks for that:
constexpr uint32_t request_chunk(int q, int lane) { return (uint32_t)((lane & 7) ^ ((q & 1) * 4 + (lane >> 4))) * 16u; }

// Where K may be an odd multiple of 32 (blocks of 32), a pair's resource starts with the pair, pair * kPairBytes into the tile's
// activations, and ends with them: a lane's own offset decides what is read, and the half line beyond the last token's end reads as
// zero.  (With the resource at the tile's start and the pair's as the scalar offset of the load that half line is kept out only by a
// range check that covers the sum of both offsets.  The one of this chip does: 64 lanes x 16 bytes read through a resource of 4096
// bytes at scalar offset 3584 give zeros from lane 32 on, 4-byte, 16-byte and LDS loads alike.)
// A pair past the end of K has an empty resource; any other starts inside the first token.
constexpr uint32_t resource_bytes(uint32_t bytes, int pair, int stages) {
    return 2 * pair < stages ? bytes - (uint32_t)pair * kPairBytes : 0u;
}

}  // namespace tman
