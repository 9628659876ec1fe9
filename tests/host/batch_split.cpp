// Prints the split of the batch pair kernels for the triples (T, tiles, slots,
// range_bytes) on standard input: ranges, their length and the modelled time.
#include <cstdio>

#include "batch_split.h"

int main() {
    int T, tiles, slots;
    long long bytes;
    while (std::scanf("%d %d %d %lld", &T, &tiles, &slots, &bytes) == 4) {
        int ns = 0, len = 0;
        bem::batch_split(T, tiles, slots, bytes, &ns, &len);
        std::printf("%d %d %.17g\n", ns, len, bem::batch_split_cost(tiles, slots, ns, len));
    }
}
