// Directed ring sum: what a reversal of the ranks i .. j, q = j + 1, adds, as one term per rank (cc_2opt_dsum_pruned.hip).  f: the hops as
// walked, b: the same edges the other way, upto: the prefix sum of b - f, turned: sum b - sum f.
#pragma once
#include <hip/hip_runtime.h>

namespace cc {
namespace dsum {

// What a move adds fits 32 bits (N hops below 2^21), one rank's term alone does not always: N = 1024, all hops as walked the largest
// cost, the other way 0, and rank j = N - 1, whose q = 0 stands in `upto` as well: -1025 (2^21 - 1).  So terms are unsigned, where
// they wrap, and so does their sum, back to what it is.
struct Terms {
    int kept, other;                        // walked as it was, and the other way
};
__host__ __device__ constexpr Terms term_of_first(int kept_least, int other_least, int f, int b, int upto) {
    return {(int)((unsigned)kept_least - (unsigned)f - (unsigned)upto), (int)((unsigned)other_least - (unsigned)b + (unsigned)upto)};
}
__host__ __device__ constexpr Terms term_of_last(int kept_least, int other_least, int f_q, int b_q, int upto, int turned) {
    return {(int)((unsigned)kept_least - (unsigned)f_q + (unsigned)upto),
            (int)((unsigned)other_least - (unsigned)b_q - (unsigned)upto + (unsigned)turned)};
}
__host__ __device__ constexpr int together(int first, int last) { return (int)((unsigned)first + (unsigned)last); }

}  // namespace dsum
}  // namespace cc
