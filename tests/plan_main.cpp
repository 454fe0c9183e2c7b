// Reads lattices (nx ny nz phase wide half cus chunk_z tile_rows state_bytes) and prints
// the plan of each: rows, z chunk, work items, store hint, launches of 1024 threads.  The first line printed holds
// the constants of the cost model.
#include <cstdio>

#include "tslb_plan.h"

int main() {
    using namespace tslb;
    std::printf("%d %.17g %.17g %lld %lld\n", kMaxChunk, kWideCost, kWideCostHalf, fused_walk2({1, 1, 1, true, true, false, 1}, 0),
                fused_walk2({1, 1, 1, false, false, false, 1}, 0));
    int nx, ny, nz, phase, wide, half, cus, chunk, rows;
    long long bytes;
    while (std::scanf("%d %d %d %d %d %d %d %d %d %lld", &nx, &ny, &nz, &phase, &wide, &half, &cus, &chunk, &rows, &bytes) == 10) {
        const PlanShape s{nx, ny, nz, phase != 0, wide != 0, half != 0, cus};
        const FusedPlan p = plan_fused(s, chunk, rows);
        const long long items = fused_tiles(s, p.rows) * chunk_count(nz, p.lz);
        long long launches = 0, first = 0;
        for (long long n; first < items; first += n, ++launches) {
            n = launch_blocks(items - first, 1024);
            if (n < 1 || n * 1024 > 0xFFFFFFFFll) return 1;
        }
        if (first != items) return 1;
        std::printf("%d %d %lld %d %lld\n", p.rows, p.lz, items, stream_stores(s, (size_t)bytes), launches);
    }
    return 0;
}
