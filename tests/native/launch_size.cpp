// The tile shapes picked for projections of very many rows keep their grids
// below 2^32 threads (the blocks that convert weights included).
#include "oc_attn_common.h"
#include "oc_ring_tile.h"
#include <cstdio>

using namespace oc;

int main() {
    constexpr int threads[N_RING_SHAPES] = {RING_THREADS<0>, RING_THREADS<1>, RING_THREADS<2>, RING_THREADS<3>,
                                            RING_THREADS<4>, RING_THREADS<5>, RING_THREADS<6>, RING_THREADS<7>,
                                            RING_THREADS<8>, RING_THREADS<9>};
    for (int hd : {16, 32, 48, 64, 128})
        for (int C : {8, 64, 320})
            for (long rows = 1L << 20; rows < 1L << 30; rows += rows / 3 + 1)
                for (int which = 0; which < 2; ++which) {
                    const auto tiles = [&](int BA, int BB) {   // Q/K/V, output
                        return which == 0 ? (long)cdiv(2 * hd, BA) * cdiv((int)rows, BB) + (long)cdiv((int)rows, BA) * cdiv(hd, BB)
                                          : (long)cdiv(C, BA) * cdiv((int)rows, BB);
                    };
                    const int K = which == 0 ? C : hd, id = ring_pick(K, tiles);
                    bool any = false;
                    for (int i = 0; i < N_RING_SHAPES; ++i)
                        any |= (tiles(RING_SHAPES[i].BA, RING_SHAPES[i].BB) + N_CUS) * threads[i] < 1L << 32;
                    const long n = (tiles(RING_SHAPES[id].BA, RING_SHAPES[id].BB) + N_CUS) * threads[id];
                    if (any && n >= 1L << 32) {
                        std::printf("%ld rows, C %d, hd %d: shape %d, %ld threads\n", rows, C, hd, id, n);
                        return 1;
                    }
                }
    return 0;
}
