// How the degrees of an edge list are counted (vertex_order_build): ids of B bits are
// parted by their top part_bits, and each part is counted by `copies` blocks, one share of
// its keys and one copy of its counts each, `range` ids at a time in LDS.
#pragma once

#include <algorithm>
#include <cstdint>

namespace dg {

constexpr int DEG_RANGE_BITS = 13, DEG_RANGE = 1 << DEG_RANGE_BITS;  // 32 KB of counts
constexpr int DEG_COPIES = 8;

struct DegreePlan {
    int part_bits, copies;
};

// A block reads its keys once per DEG_RANGE ids of its part (64M keys: 84 us), and eight
// more bits of parting are one more pass of the sort (500 us).  So up to 24 bits one pass and
// up to eight reads are as good as two passes and one; from 25 bits on two passes keep the
// reads at one (two at the largest n), where one pass read 2^(B - 21) times: building 2^26
// vertices and 64M arcs 21.9 ms of kernels with one pass, 19.6 with two, 2^28 vertices
// 50.9 and 39.8.
// Copies spread the keys of a part that holds many of them; each costs 8 bytes of traffic
// and 4 of memory per id, so graphs of few arcs a vertex take fewer, and no more memory than
// the rows of the built graph will.
inline DegreePlan degree_plan(int B, int64_t n, int64_t arcs) {
    DegreePlan p;
    p.part_bits = B <= 24 ? std::min(B, 8) : std::min(B - DEG_RANGE_BITS, 16);
    p.copies = (int)std::min<int64_t>(DEG_COPIES, std::max<int64_t>(2, 2 * arcs / std::max<int64_t>(n, 1)));
    return p;
}

}  // namespace dg
