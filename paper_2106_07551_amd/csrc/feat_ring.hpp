// The order in which a wavefront of the feature step reads W's operand blocks,
// in plain C++ so that it can be followed on the host.
#pragma once

namespace malib {

// W packed for a state of d = 16 kg values: kg tiles of 16 outputs, each kg blocks
// of 16 inputs, kg * kg blocks in all.
constexpr int feat_block(int tile, int group, int kg) { return tile * kg + group; }

// A ring of `depth` slots (a divisor of kg) holds groups g0 .. g0 + depth - 1 at the
// start of the round at g0; whether the round refills its slots, with the groups
// depth later.  The last round does not: those would be the next tile's blocks and,
// from the last tile on, lie outside W.
constexpr bool feat_refills(int g0, int depth, int kg) { return g0 + depth < kg; }

}  // namespace malib
