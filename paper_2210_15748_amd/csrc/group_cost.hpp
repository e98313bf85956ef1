// What an assignment by groups of centroids (filter_groups.hip) costs against comparing every vector with every centroid, and when it is
// done (constexpr: for the kernels and, without HIP, for the host).
#pragma once
#include <stdint.h>

namespace dessert {

constexpr uint32_t GROUP_TRIAL = 4096;   // vectors that tell whether the groups pay
struct GroupCtl {   // what the launches of an assignment tell each other
    uint32_t groups;    // groups of centroids
    uint32_t radius2;   // largest squared distance of a centroid from its group's leader
    uint32_t easy;      // vectors of the trial that need one group only
    uint32_t members;   // centroids in the groups of those, added up
    uint32_t rest;      // vectors left to a comparison with every centroid
    uint32_t led;       // centroids that have looked for their leader before the others, and
    uint32_t alone;     // those of them that lead themselves
    uint32_t skip;      // != 0: not tried
};
constexpr uint32_t groups_room(uint32_t K) { return K / 3; }   // more groups are not made
// Of a vector, in products of a vector and a centroid as the comparison with every centroid makes them (on the matrix cores, rows shared by 512
// vectors): a member of its group costs 56 to 80 of them (rows from L2 for each vector; 500 000 vectors, 16 384 centroids around 128, 256 and 512
// centres, d = 128 62, 68 and 72, d = 256 56, 66 and 70), a leader 1.2, a vector that is left over all of them again and something for its list.
constexpr uint32_t GROUP_MEMBER = 75;
constexpr uint32_t groups_largest(uint32_t K) { return K / GROUP_MEMBER; }   // a vector of a larger group is left over
// The trial's vectors by groups against all of their products.  0.9: what the estimate is good to.  Mixtures of 64 centres, 16 384 centroids
// (256 members to a group), 1.24 of the time of comparing with all where the members were not counted.
constexpr bool groups_pay(const GroupCtl& c, uint32_t K) {
    if (c.groups == 0 || c.groups > groups_room(K)) return false;
    const uint64_t all = (uint64_t)GROUP_TRIAL * K;
    const uint64_t tenths = 12ull * GROUP_TRIAL * c.groups + 10ull * GROUP_MEMBER * c.members + 11ull * (GROUP_TRIAL - c.easy) * K;
    return tenths <= 9 * all;
}

// The search for leaders makes up to K * K / 2 products, at a worse rate than a comparison with every centroid.  From GROUP_MANY centroids on some
// of them, spread evenly, look first: where so many lead themselves there will be about as many groups as are made at most, and no others look.
// (600 000 vectors, 65 536 centroids around 30 000 centres, d = 256: 1.24 of the time of comparing with all without it, 1.04 with.)
constexpr uint32_t GROUP_MANY = 32768;
constexpr uint32_t GROUP_LOOKS = 128;   // workgroups
constexpr bool groups_hopeless(uint32_t led, uint32_t alone) { return (uint64_t)alone * 10 > (uint64_t)led * 3; }
// Rounds of k-means: where the groups of one did not pay, those of the next are not made.  Of every eight the first two always try: after the
// first the centroids are means instead of vectors, which can change what pays.
constexpr bool group_round_tries(uint32_t round) { return round % 8 < 2; }

}  // namespace dessert
