// Loads that may still be under way at the counted waits of the tall tiles (matmul_a8_tiled128.hip, matmul_a16_fold.hip): no HIP, so
// that a test can compile it by itself.
//
// Stage s asks for the activations of stage s + ahead; the first stage of a 256-k tile asks for the next tile's weights and scales
// before that.  With pairs of stages (eight buffers) a barrier stands behind every second stage, and the pair behind it reads up to its
// third stage; else (four buffers) behind every stage, and the next one reads two.  Vector memory operations complete in order.
#pragma once

namespace w2 {

namespace tall {

constexpr int ahead(bool pair) { return pair ? 6 : 3; }

// before the first stage.  np: a wave's loads of activations per stage
constexpr int at_start(bool pair, int np) { return (ahead(pair) - (pair ? 3 : 2)) * np; }

// behind stage t of a tile (pairs: odd ones).  w: loads of weights and scales counted on per tile
constexpr int behind(bool pair, int t, int np, int w) { return pair ? 3 * np + (t == 1 ? w : 0) : np + (t == 0 ? w : 0); }

// One of each per column block.  An export of the group sums reads no scale and the compiler drops those loads: it counts on none
// (fewer counted than issued only waits for more).
constexpr int weights(bool exported, int cj) { return exported ? 0 : 2 * cj; }

}  // namespace tall

}  // namespace w2
