// The worker pass's items on the host, with the functions its kernel and
// launcher use: the division that splits an item into row and block is exact
// for every divisor and item below 2^31, and the pieces of a call take every
// (row, block) once.  Exit status 0 when every case passes.
#include "onebit_grid.h"

#include <cstdio>
#include <vector>

using namespace onebit;

static int failures = 0;

static void check_quotient(int64_t d, int64_t x)
{
    if (x < 0 || x >= ((int64_t)1 << 31)) return;
    if (fast_quotient(x, fast_div(d)) != x / d && failures++ < 20)
        std::printf("FAIL %lld / %lld\n", (long long)x, (long long)d);
}

// rows x blocks items in pieces of at most `piece` items, one workgroup each.
static void check_pieces(int64_t rows, int64_t blocks, int64_t piece)
{
    const int64_t items = rows * blocks;
    const FastDiv by = fast_div(blocks);
    std::vector<unsigned char> seen((size_t)items, 0);
    for (int64_t base = 0; base < items; base += piece) {
        const int64_t count = items - base < piece ? items - base : piece;
        const int64_t grid = xcd_grid(count, 1);
        for (int64_t b = 0; b < grid; ++b) {
            const int64_t at = xcd_block_of(b, grid);
            if (at >= count) continue;
            const int64_t item = base + at;
            const int64_t i = fast_quotient(item, by), blk = item - i * blocks;
            if (i < 0 || i >= rows || blk < 0 || blk >= blocks || seen[(size_t)item]++)
                if (failures++ < 20) std::printf("FAIL item %lld\n", (long long)item);
        }
    }
    for (int64_t k = 0; k < items; ++k)
        if (!seen[(size_t)k] && failures++ < 20) std::printf("FAIL item %lld left out\n", (long long)k);
}

int main()
{
    const int64_t top = ((int64_t)1 << 31) - 1;
    std::vector<int64_t> divisors;
    for (int64_t d = 1; d <= 3000; ++d) divisors.push_back(d);
    for (int s = 11; s <= 30; ++s)
        for (int64_t k = -3; k <= 3; ++k) divisors.push_back(((int64_t)1 << s) + k);
    for (int64_t d : {106337ll, 326258ll, 527431ll, 4194307ll, 33554393ll, (long long)top}) divisors.push_back(d);
    for (int64_t d : divisors) {
        // both sides of multiples of d, near 0, in the middle and near 2^31
        for (int64_t q : {(int64_t)0, (int64_t)1, (int64_t)2, top / d / 3, top / d / 2, top / d - 1, top / d})
            for (int64_t k = -2; k <= 2; ++k) check_quotient(d, q * d + k);
        check_quotient(d, top);
    }
    for (int64_t rows : {1, 2, 3, 8, 33})
        for (int64_t blocks : {1, 2, 7, 64, 1023, 3001}) {
            check_pieces(rows, blocks, 1 << 20);
            check_pieces(rows, blocks, 24);
            check_pieces(rows, blocks, 1000);
        }
    if (failures) return 1;
    std::printf("items_check: ok\n");
    return 0;
}
