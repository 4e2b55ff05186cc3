// Which K-steps the rings of head_once_kernel hold when.  For the kernel, and for a test on the host that goes through them.
#pragma once

namespace specdraft {

constexpr int kOnceDW = 8;         // K-steps (of 32) of weights in LDS
constexpr int kOnceDS = 4;         // and of states

// The step that goes into slot (step % depth) of a ring of `depth` slots once `step` has been read from it: the one `depth` steps on.
// Past the end of K the last step again: nobody reads it, it is in the L2, and it lies in the matrix.
constexpr int once_next_step(int step, int depth, int kt) { return step + depth < kt ? step + depth : kt - 1; }

}  // namespace specdraft
