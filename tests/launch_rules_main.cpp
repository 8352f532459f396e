// The launch rules of the library (csrc/launch_rules.h) on the CPU.
#include <cstdio>
#include <initializer_list>
#include "launch_rules.h"

// The projection of few rows reads U (d x k) NB floats a lane, 32 rows a tile: no unguarded load may pass its end.
static int check_unguarded_tiles() {
    for (int nb : {2, 4})
        for (int d = 256; d <= 352; ++d)
            for (int k = 1; k <= 40; ++k) {
                const int n = splc::unguarded_tiles(d, k, nb, 32);
                if (n < 0 || n > d / 32 || (k % nb == 0 && n != d / 32) || n < d / 32 - 1) {
                    printf("d %d k %d nb %d: %d tiles\n", d, k, nb, n);
                    return 1;
                }
                for (int row = 0; row < 32 * n; ++row)
                    for (int col = 0; col < k + nb; col += nb) {
                        const long first = (long)row * k + (col < k ? col : 0);
                        if (first + nb > (long)d * k) {
                            printf("d %d k %d nb %d: row %d column %d reads element %ld of %ld\n", d, k, nb, row, col,
                                   first + nb - 1, (long)d * k);
                            return 1;
                        }
                    }
            }
    return 0;
}

int main() {
    if (check_unguarded_tiles()) return 1;
    printf("ok\n");
    return 0;
}
