// Launch sizes that follow from a call's sizes alone (host only, no HIP).
#pragma once

#include <stdint.h>

namespace ptsd {

// Bytes of a copy unit's usual chunk: what a block is worth is counted in them.
constexpr int64_t kPieceBytes = 32 << 10;

// Workgroups of a scatter of up to `entries` blocks: `units` units and `bytes`
// bytes of each are moved; `round` workgroups fill the device. They loop over
// the units. The host does not know how few blocks were created, so a scatter
// of a few blocks pays for the workgroups that find nothing, and one of very
// many for too few that loop:
//
//   workgroups                       512   1,024  2,048  4,096  8,192
//   64 of 4,096 blocks of 128 KiB   10.1   10.1   10.0   11.0   14.0 us
//   all of them                    214.6  212.7  210.7  207.4  205.9
//   4 of 256 blocks of 2 MiB        10.0   10.2   10.1   11.0   13.9
//   all of them                    202.2  197.9  195.4  192.6  190.0
//   all of 512 blocks of 1.25 MiB,
//   units of 256 KiB               281.4  279.1  275.9  269.9  269.9
//
// Four rounds cost a sparse call nothing; past that the grid follows what a
// block is worth and what the call could move at all, up to 16 rounds (five
// units of 256 KiB are worth forty of 32 KiB, not five). One layer of the 8B
// shape, 7,168 blocks, takes 156.7 us by this rule and 155.8 at 16 rounds.
inline int64_t scatter_grid(int64_t round, int64_t entries, int64_t units, int64_t bytes) {
    int64_t pieces = bytes / kPieceBytes > units ? bytes / kPieceBytes : units;
    if (pieces > 1 << 20) pieces = 1 << 20;  // far past 16 rounds; keeps the products in 64 bits
    const int64_t reach = entries * pieces / 4;
    int64_t g = round * pieces < reach ? round * pieces : reach;
    if (g < 4 * round) g = 4 * round;
    if (g > 16 * round) g = 16 * round;
    return g < entries * units ? g : entries * units;
}

}  // namespace ptsd
