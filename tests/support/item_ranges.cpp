// Reads "spp log2" lines and prints, for each, the first item of a ray's 2^log2
// work items whose sample range does not follow the one before it (items must
// cover 0 .. spp in order, none empty), or -1.  Built on the host only.
#include "../../paper_1903_03837_amd/csrc/tracer_device.hpp"
#include <cstdio>

int main() {
    int spp, log2;
    while (std::scanf("%d %d", &spp, &log2) == 2) {
        const long long items = 1ll << log2;
        long long bad = lp::item_sample(0, spp, log2) == 0 ? -1 : 0;
        for (long long i = 0; i < items && bad < 0; ++i) {
            const int a = lp::item_sample((int)i, spp, log2), b = lp::item_sample((int)i + 1, spp, log2);
            if (!(0 <= a && a < b && b <= spp)) bad = i;
        }
        if (bad < 0 && lp::item_sample((int)items, spp, log2) != spp) bad = items;
        std::printf("%lld\n", bad);
    }
    return 0;
}
