/* Answers what csrc/bl_gemm_choice.h chooses: one question a line on stdin, one answer a line on stdout.
 *   plain M N K residual acc y  place of the kernel (5: the split k loop)
 *   residual M N K | gate M N K   place of the tile
 *   stores M N acc              whether fp32 output is stored past the caches
 *   order M N                   the split k loop's order: across, bytes per k that an XCD reads
 *   table entries steps chain   whether a table of 33 to 48 tokens goes to the tile kernel
 *   tiles tiles_m tiles_n BM K  the tile kernels' order: gm, band, vgrid */
#include "bl_gemm_choice.h"

#include <stdio.h>
#include <string.h>

int main() {
    char what[16];
    while (scanf("%15s", what) == 1) {
        int a, b, c, d, e, f;
        if (!strcmp(what, "plain") && scanf("%d %d %d %d %d %d", &a, &b, &c, &d, &e, &f) == 6) {
            printf("%d\n", bl_plain_kernel(a, b, c, d != 0, e != 0, f != 0));
        } else if (!strcmp(what, "residual") && scanf("%d %d %d", &a, &b, &c) == 3) {
            printf("%d\n", bl_residual_kernel(a, b, c));
        } else if (!strcmp(what, "gate") && scanf("%d %d %d", &a, &b, &c) == 3) {
            printf("%d\n", bl_gate_kernel(a, b, c));
        } else if (!strcmp(what, "stores") && scanf("%d %d %d", &a, &b, &c) == 3) {
            printf("%d\n", (int)bl_past_caches(a, b, c != 0));
        } else if (!strcmp(what, "table") && scanf("%d %d %d", &a, &b, &c) == 3) {
            printf("%d\n", (int)bl_table_in_tiles(a, b, c));
        } else if (!strcmp(what, "order") && scanf("%d %d", &a, &b) == 2) {
            const bl_ksplit_order o = bl_ksplit_order_of(a, b);
            printf("%d %lld\n", (int)o.across, (long long)o.bytes);
        } else if (!strcmp(what, "tiles") && scanf("%d %d %d %d", &a, &b, &c, &d) == 4) {
            const bl_tile_order o = bl_tile_order_of(a, b, c, d);
            printf("%d %d %d\n", o.gm, o.band, o.vgrid);
        } else {
            return 1;
        }
    }
    return 0;
}
