// Host check of the grid of the short-K ring kernel (ring_grid.h): every step has a walker, and no XCD gets more workgroups
// than its 32 CUs hold together, as long as the sets of column groups leave that possible.
#include <cstdio>

#include "../../paper_1806_08342_amd/csrc/ring_grid.h"

int main()
{
    for (int per_cu = 1; per_cu <= 4; ++per_cu)
        for (int sets = 1; sets <= 300; ++sets)
            for (int steps = 1; steps <= 40000; steps += steps < 600 ? 1 : 997) {
                const int w = qnn::ring_walkers(per_cu, sets, steps);
                const int most = (w + 7) / 8 * sets; // workgroups of the fullest XCD
                const bool fits = sets > 32 * per_cu || most <= 32 * per_cu;
                if (w < 1 || w > steps || !fits) {
                    std::printf("per_cu %d sets %d steps %d: %d walkers, %d workgroups on one XCD\n", per_cu, sets, steps, w, most);
                    return 1;
                }
            }
    return 0;
}
