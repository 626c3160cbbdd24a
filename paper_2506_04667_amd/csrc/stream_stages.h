// Which stage of the activations' LDS ring the weight-streaming kernels' epilogue goes through.  Plain C++, so that the order of reads, copies
// and barriers can be replayed on the host around the rule that the kernels use.
#pragma once

namespace moe {

// Pair q of K-tiles is multiplied out of stage q % stages.
constexpr int stream_next_stage(int stage, int stages) { return stage + 1 == stages ? 0 : stage + 1; }

// A wavefront stages its output rows in its own eighth of a stage (where its own copies go and no other's) that nobody reads any more and that no
// copy in flight writes, after the pair in stage `sa`:
//   two stages in the ring: the third one, which nothing else uses;
//   three, and more pairs follow: sa.  The barrier in the pair's odd tile comes after everybody's last read of it; the next copies into a
//     wavefront's eighth are its own and issued after its stores, which need what it read back;
//   three, and the stream ends (`last`): that tile has no barrier, others may still be reading sa.  The stage after it was read for the last
//     time two pairs ago, no copy of a pair beyond the stream's end was requested, and all copies had landed at the barrier in the even tile.
constexpr int stream_epilogue_stage(int stages, int sa, bool last) { return stages == 2 ? 2 : last ? stream_next_stage(sa, stages) : sa; }

}  // namespace moe
