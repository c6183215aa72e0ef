// Plays where the waves of a team leave a part (csrc/attn_division.h, PartRegion; csrc/attn_parts.h): every store of every lane, for 64
// and 128 columns, 1 .. 4 waves that share the columns, row tiles of 32 .. 256 rows.  Prints the first store that leaves the region
// or overlaps another one, exit status 1.
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include <vector>

#include "attn_division.h"

using namespace s4c;

template <int D>
static void play(int M, int keys, int tile_rows) {
    typedef PartRegion<D> R;
    std::vector<char> used(R::bytes(M), 0);
    auto store = [&](uint32_t at, int bytes, const char* what) {
        for (int i = 0; i < bytes; ++i)
            if (at + i >= used.size() || used[at + i]++ || at % (bytes < 16 ? 8 : 16)) {
                printf("%d rows, %d columns, %d waves, tiles of %d: %s at %u\n", M, D, keys, tile_rows, what, at);
                exit(1);
            }
    };
    const int blocks = (M + 31) / 32;
    for (int block = 0; block < blocks; ++block)
        for (int key = 0; key < keys; ++key)
            for (int lane = 0; lane < 64; ++lane) {
                if (32 * block + lane % 32 >= M) continue;
                for (int q = 0; q < D / 8 / keys; ++q) store(R::slab(M, block, key * (D / 8 / keys) + q, lane), 16, "a slab");
                if (lane < 32) store(R::stats(M, block, key, lane), 8, "a row's statistics");
            }
    for (int mt = 0; mt < (M + tile_rows - 1) / tile_rows; ++mt) store(R::word(M, mt), 8, "a word");
    long n = 0;
    for (char c : used) n += c;
    if (n != 4l * M * D + 8l * keys * M + 8l * ((M + tile_rows - 1) / tile_rows)) {
        printf("%d rows, %d columns: something is missing\n", M, D);
        exit(1);
    }
}

int main() {
    for (int M = 1; M <= 2048; M += M < 300 ? 1 : 61)
        for (int tile : {32, 64, 128, 256})
            for (int keys : {1, 2, 4}) {
                if (keys < 4) play<64>(M, keys, tile);
                play<128>(M, keys, tile);
            }
    return 0;
}
