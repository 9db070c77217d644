// Simulates on the host which positions of the Vt rows the projection's tiles
// write (the rules of oc_attn_common.h and the tile shapes of oc_ring_tile.h)
// and reports the first call whose key padding is read but not covered.
//   vt_cover                             every tile shape over a grid of batches
//   vt_cover heads dh C n_seq L n_ctx    tile rows, positions its tiles cover, lpad, and whether the DMA attention follows
#include "oc_attn_common.h"
#include "oc_ring_tile.h"
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

using namespace oc;

// first position of [0, lpad) that no write of a sequence covers, -1 if none
static int uncovered(int BA, int n_seq, int L, int Lk, int lpad, bool zero_pad) {
    std::vector<char> w(lpad, 0);
    if (vt_whole_rows(n_seq, L, BA)) {
        for (int j0 = 0; j0 < Lk; j0 += BA)
            for (int j = j0; j < vt_tile_end(j0, BA, Lk, lpad); ++j) w[j] = 1;
    } else {
        for (int j = 0; j < (zero_pad ? lpad : Lk); ++j) w[j] = 1;   // tokens, then the zeroed padding
    }
    for (int j = 0; j < lpad; ++j)
        if (!w[j]) return j;
    return -1;
}

int main(int argc, char **argv) {
    if (argc == 7) {
        int v[6];
        for (int i = 0; i < 6; ++i) v[i] = std::atoi(argv[i + 1]);
        Plan p;
        AttnArgs a;
        std::memset(&p, 0, sizeof(p));
        std::memset(&a, 0, sizeof(a));
        p.heads = v[0]; p.dh = v[1]; p.hd = v[0] * v[1]; p.C = v[2]; p.n_ctx = v[5]; p.bf16 = true; p.esz = 2;
        a.n_seq = v[3]; a.L = v[4];
        const int rows = a.n_seq * a.L + p.n_ctx, Lk = a.n_seq == 1 ? rows : a.L;
        const int id = ring_pick(p.C, [&](int BA, int BB) {
            return (long)cdiv(2 * p.hd, BA) * cdiv(rows, BB) + (long)cdiv(rows, BA) * cdiv(p.hd, BB);
        });
        const int BA = RING_SHAPES[id].BA;
        std::printf("%d %d %d %d\n", BA, vt_whole_rows(a.n_seq, a.L, BA) ? cdiv(Lk, BA) * BA : -1,
                    attn_ws(p, a.n_seq, a.L, 0).lpad,
                    !attn_short(Lk) && !flash_splits(p, a, Lk) && flash_uses_dma(p.dh, Lk, p.hd) ? 1 : 0);
        return 0;
    }
    for (const RingShapeCost &c : RING_SHAPES)
        for (int heads : {1, 64})   // the keys shared out / staged by DMA
            for (int n_seq : {1, 2, 7})
                for (int L = 65; L <= 2500; ++L)
                    for (int n_ctx : {0, 77}) {
                        if (n_seq > 1 && n_ctx > 0) continue;
                        Plan p;
                        AttnArgs a;
                        std::memset(&p, 0, sizeof(p));
                        std::memset(&a, 0, sizeof(a));
                        p.heads = heads; p.dh = 64; p.hd = heads * 64; p.C = 64; p.n_ctx = n_ctx; p.bf16 = true; p.esz = 2;
                        a.n_seq = n_seq; a.L = L;
                        const int Lk = n_seq == 1 ? L + n_ctx : L, lpad = attn_ws(p, n_seq, L, 0).lpad;
                        const bool read = vt_padding_read(p, a, Lk);
                        const int at = uncovered(c.BA, n_seq, L, Lk, lpad, read);
                        if (read && at >= 0) {
                            std::printf("tile of %d rows, %d heads, %d x %d + %d: position %d of %d\n", c.BA, heads, n_seq, L,
                                        n_ctx, at, lpad);
                            return 1;
                        }
                    }
    return 0;
}
