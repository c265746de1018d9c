// The residual cache's bounds on the host, for the kernels' row layouts: reads vocabulary
// sizes from argv and, for each layout, walks every slot and chunk that a pass visits.  The
// chunks that rc_holds admits must lie in the sequence's half of the cache and hold the
// whole row.  Prints "V surplus" per size: how many visited elements the cache does not hold
// (the largest over the layouts).
#include <cstdio>
#include <cstdlib>

#include "common.h"

template <int VEC, int UNR>
long check(int V) {
    constexpr int CHUNK = 64 * VEC * UNR;
    const SlotLayout l = slot_layout<VEC, UNR>(V);
    const long half = rc_half(V);
    long held = 0, surplus = 0;
    for (int s = 0; s < l.nslots; ++s) {
        // the passes that read the cache take the first n chunks of a slot
        const int n = rc_slot_chunks(s, l.G, CHUNK, (int)half);
        if (n < 1 || n > l.G) return -4;
        for (int j = 0; j < l.G; ++j) {
            const int c0 = (s * l.G + j) * CHUNK;
            for (int u = 0; u < UNR; ++u) {
                // one load: elements [i0, i0 + 64 * VEC), taken or left as a whole
                const int i0 = c0 + u * 64 * VEC;
                if (rc_holds(i0, (int)half) != (j < n)) return -5;
                if (rc_holds(i0, (int)half) != rc_holds(c0, (int)half)) return -1;
                if (!rc_holds(i0, (int)half)) {
                    surplus += 64 * VEC;
                    continue;
                }
                if (i0 + 64 * VEC > half) return -2;
                held += 64 * VEC;
            }
        }
    }
    return held >= V ? surplus : -3;
}

int main(int argc, char** argv) {
    for (int k = 1; k < argc; ++k) {
        const int V = atoi(argv[k]);
        const long got[3] = {check<8, kUnr16>(V), check<4, kUnr32>(V), check<1, 4>(V)};
        long most = 0;
        for (const long g : got) {
            if (g < 0) {
                printf("%d fails %ld\n", V, g);
                return 1;
            }
            most = g > most ? g : most;
        }
        printf("%d %ld\n", V, most);
    }
    return 0;
}
