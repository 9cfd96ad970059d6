// How many passes the host asks for before it looks again, where the device goes from update to update of the initialisation by itself
// (host only; see walk in rb_derive.hip)
#pragma once
#include <algorithm>

namespace rb {
namespace derive {

constexpr int FIRST_LOOK = 4;          // power iterations before the first look
constexpr int MOST_PASSES = 1024;      // passes asked for without a look

// What a look tells: passes asked for so far, those of them that went into the update under way, updates that are finished and those that are left.
// As many as the rest would take at the mean so far and two more: they (some 6 us each) are less than another look (27 us).
// But updates take a few iterations mostly and two hundred at most, and one of them says little of the others (after a first one of 200 the mean
// asked for 900 passes that had nothing to do, and for two at a time in a slow one after quick ones).  So no more than FIRST_LOOK + 1 iterations for each
// update, but a quarter of what the one under way has taken, or an eighth of all, in any case: a look, or passes too many, cost little beside that.  (While none is
// finished FIRST_LOOK at a time: one path of 1024 x 2048, an update of five iterations, 220 us where two take 180)
inline int passes_to_ask(double passes, double under_way, double finished, double left)
{
    double n = 2.0;
    if (finished > 0.0) n = std::min((FIRST_LOOK + 2) * left, std::max(0.0, (passes - under_way) / finished * left - under_way) + 2.0);
    return (int)std::min<double>(MOST_PASSES, std::max(n, std::max(passes / 8.0, under_way / 4.0)));
}

}  // namespace derive
}  // namespace rb
