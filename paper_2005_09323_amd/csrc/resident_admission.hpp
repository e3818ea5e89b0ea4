// Which resident launches of one process may run on the device together.
// (Host code without HIP.)
#pragma once

#include <algorithm>
#include <vector>

namespace lbm {

// What a context's launches that may be running take of the device: the most
// workgroups of any of them, and how many of these a compute unit holds (0:
// they differ in that; they run beside no other context's).
struct ResidentUse {
    int blocks = 0, places = 1;
};

// A context's use where launches of both kinds may be running, one at a time.
inline ResidentUse either_of(const ResidentUse& a, const ResidentUse& b) {
    ResidentUse u;
    u.blocks = std::max(a.blocks, b.blocks);
    u.places = a.places == b.places ? a.places : 0;
    return u;
}

// True if every workgroup of one launch of each context is on the device at
// the same time, whatever the order they are dispatched in.
inline bool side_by_side(const std::vector<ResidentUse>& uses, int compute_units) {
    long long blocks = 0;
    for (const ResidentUse& u : uses) {
        if (uses.size() > 1 && (u.places == 0 || u.places != uses[0].places)) return false;
        blocks += u.blocks;
    }
    return uses.size() < 2 || blocks <= (long long)compute_units * uses[0].places;
}

}  // namespace lbm
