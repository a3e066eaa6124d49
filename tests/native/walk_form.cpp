// Prints the walk form of packed headers: per line of standard input the
// layout, bytes of a block, classes, used features and bytes of the node
// section.
#include <cstdio>

#include "fp_internal.h"

int main() {
    long long layout, block, classes, used, section;
    while (scanf("%lld %lld %lld %lld %lld", &layout, &block, &classes, &used, &section) == 5) {
        fp::Header h{};
        h.layout = (int32_t)layout;
        h.block_bytes = (int32_t)block;
        h.n_classes = (int32_t)classes;
        h.n_used_features = (int32_t)used;
        h.nodes_offset = 4096;
        h.total_bytes = 4096 + section;
        printf("%d\n", (int)fp::walk_form(h));
    }
    return 0;
}
