// Host replay of the network kernels' reads of a tile's rows
// (paper_2008_11520_amd/csrc/net_index.h, the functions the kernels call), with
// the thread counts, tile heights and input widths that the kernels are built
// for:
//   k_net_reg   64 rows, 8 H threads, predicated (tile_piece_in);
//   k_net_q8p   32 rows, 4 H threads, predicated; a 64-patch row tile of the
//               batch table is two such tiles, the second with rows - 32 rows
//               (none or negative for a short row tile);
//   k_net_wide  64 rows (K <= 2) or 32 (K = 3, halves as above), 4 H threads,
//               clamped (tile_piece, tile_row);
//   k_net       64 or 16 rows, clamped (tile_piece_last, tile_row).
// For every row count of a 64-patch row tile every read must lie inside the row
// tile's rows, and every row whose results are stored must receive its own
// pieces, once.
#include "net_index.h"

#include <climits>
#include <cstdio>
#include <vector>

using namespace dnnmg;

static int fails = 0;
static long reads = 0;
static void check(bool ok, const char *what, int rows, int c)
{
    if (!ok && fails++ < 10) std::printf("FAIL: %s, %d rows, piece or row %d\n", what, rows, c);
}

// One tile of R rows, threads NT, per_row pieces per row, starting at row `at` of
// a row tile of `rows` rows.  read(c, nrows) is the piece read for piece c, or INT_MIN.
template <typename Read>
static void tile(const char *what, int R, int NT, int per_row, int at, int rows, Read read)
{
    const int pieces = R * per_row, nrows = min(R, rows - at);
    std::vector<int> seen(pieces, 0);
    for (int t = 0; t < NT; ++t)
        for (int c = t; c < (pieces + NT - 1) / NT * NT; c += NT) {
            const int p = read(c, nrows);
            if (p == INT_MIN) continue;                                // predicated off
            const int q = at * per_row + p;                              // in the row tile
            check(q >= 0 && q < rows * per_row, what, rows, c);
            ++reads;
            if (c < pieces && c / per_row < nrows) {
                check(p == c, what, rows, c);
                ++seen[c];
            }
        }
    for (int c = 0; c < nrows * per_row; ++c) check(seen[c] == 1, what, rows, c);
}

static void predicated(const char *what, int R, int NT, int per_row)
{
    for (int rows = 1; rows <= 64; ++rows)
        for (int at = 0; at < 64; at += R)
            tile(what, R, NT, per_row, at, rows, [&](int c, int nrows) {
                return tile_piece_in(c, per_row, nrows) ? c : INT_MIN;
            });
}

// The state in the update's lane layout: rows 16 q + l.
static void state_rows(const char *what, int R)
{
    for (int rows = 1; rows <= 64; ++rows)
        for (int at = 0; at < 64 && (R != 16 || at < rows); at += R) {
            const int nrows = min(R, rows - at);
            for (int r = 0; r < R; ++r) {
                const int q = at + tile_row(r, nrows);
                check(q >= 0 && q < rows, what, rows, r);
                if (r < nrows) check(q == at + r, what, rows, r);
                ++reads;
            }
        }
}

int main()
{
    for (int H : {32, 64, 96}) {
        for (int nin : {40, 56, 104}) predicated("k_net_reg input", 64, 8 * H, nin / 8);
        predicated("k_net_reg state", 64, 8 * H, H / 4);
    }
    for (int K = 1; K <= 3; ++K) {
        const int n = 1 << K, nin = 4 * (n + 1) * (n + 1) + 4;
        for (int H : {64, 128}) {
            predicated("k_net_q8p input", 32, 4 * H, (nin + 31) / 32 * 32 / 16);
            predicated("k_net_q8p state", 32, 4 * H, H / 4);
            const int R = K <= 2 ? 64 : 32, XP = nin / 8;
            for (int rows = 1; rows <= 64; ++rows)
                for (int at = 0; at < 64; at += R)
                    tile("k_net_wide input", R, 4 * H, XP, at, rows, [&](int c, int nrows) { return tile_piece(c, XP, nrows); });
            state_rows("k_net_wide state", R);
        }
    }
    // FP32 rows (4 values a piece) and BF16 rows (8), the standard and the
    // paper's input; a flow's last tile has 1 .. R rows
    for (int V : {4, 8})
        for (int nin : {40, 104, 328, 56, 272})
            for (int H : {32, 64, 96, 128})
                for (int R : {16, 64}) {
                    const int waves = R < 64 ? H / 16 : (H == 96 ? 12 : (H < 64 ? 4 : H / 16)), per_row = nin / V;
                    for (int rows = 1; rows <= R; ++rows)
                        tile("k_net input", R, 64 * waves, per_row, 0, rows, [&](int c, int nrows) {
                            return (int)tile_piece_last((unsigned)c, (unsigned)(nrows * per_row));
                        });
                    state_rows("k_net state", R);
                }
    std::printf("%ld reads replayed, %d violations\n", reads, fails);
    return fails ? 1 : 0;
}
