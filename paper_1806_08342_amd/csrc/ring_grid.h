// Workgroups of the short-K ring kernel that share a set of column groups (host code).
#pragma once

namespace qnn {

// As many as stay resident together, `per_cu` workgroups on each of 256 CUs shared out over the sets.  The sets of a walker run on one XCD and walkers go round the eight, so each XCD
// gets the same number: 85 walkers of three sets, one workgroup per CU, put a 33rd on the 32 CUs of five XCDs, which then took
// a second round (us before and after, with the add: 26310 x 640 x 208 35.5 and 24.2, 20252 x 1552 x 176 47.2 and 31.9; without:
// 932449 x 272 x 64 148 and 123, 374564 x 832 x 192 215 and 180, 35024 x 1225 x 240 63.2 and 52.8).
inline int ring_resident(int per_cu, int sets)
{
    const int walkers = 256 * per_cu / sets / 8 * 8;
    return walkers < 8 ? 8 : walkers;
}

// ... trimmed so that every one walks the same number of the `steps` (to one)
inline int ring_walkers(int per_cu, int sets, int steps)
{
    int walkers = ring_resident(per_cu, sets);
    walkers = walkers > steps ? steps : walkers;
    const int per_walker = (steps + walkers - 1) / walkers;
    return (steps + per_walker - 1) / per_walker;
}

} // namespace qnn
