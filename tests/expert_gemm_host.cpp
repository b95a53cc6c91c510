// Host build of arithmetic that the expert GEMM kernels share with the CPU: checks by name, a line of counts each.
// Compiled and run by test_expert_gemm_host.py.
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "expert_gemm_kernel.h"

using namespace moe::gemm;

// The bounds of the buffer that a wavefront of the large tiles stores through, for every width that this kernel takes
// at a reduction of K: its rows inside the tile, in 64 bits.
static long store_bounds(int K) {
    long checked = 0;
    const int widths[] = {256, 4096, 6144, (1 << 21) + 256, 1 << 22, (1 << 22) + 512, 5592320, 5592576, (1 << 23) - 256};
    for (const int N : widths) {
        if (!offsets_fit_1w(N, K)) continue;
        for (const int esz : {2, 4})
            for (const int wave_rows : {64, 80, 96, 112, 128})
                for (const int first : {0, wave_rows})
                    for (int rows = 0; rows <= 2 * wave_rows; ++rows) {
                        const unsigned long long row_bytes = static_cast<unsigned long long>(N) * esz;
                        const int own = rows < first ? 0 : rows - first < wave_rows ? rows - first : wave_rows;
                        const unsigned long long want = own * row_bytes, last = wave_rows * row_bytes;
                        if (last >= 1ull << 32 || store_bytes(rows - first, wave_rows, row_bytes) != want) {
                            std::printf("N=%d K=%d bytes=%d rows %d of %d from %d\n", N, K, esz, rows, wave_rows, first);
                            return -1;
                        }
                        ++checked;
                    }
    }
    return checked;
}

// The map of an expert's tiles: whole tiles cover every row of every n-tile once, the halves of a tile its rows, and
// what the map names a tile has rows; a lower half without any is kEmptySlot.
static long tiles() {
    constexpr int BM = 256, NT = 3, ROW0 = 1000;
    long checked = 0;
    for (const Cut cut : {Cut::kNever, Cut::kLong, Cut::kAlways})
        for (int m_e = 1; m_e <= 2700; ++m_e) {
            static int seen[NT][2700];
            std::memset(seen, 0, sizeof(seen));
            const int mt = (m_e + BM - 1) / BM;
            for (int local = 0; local < mt * NT; ++local) {
                const TileCoord t = tile_in_expert<BM>(5, ROW0, m_e, local, NT, -1, cut);
                const int first = t.row0 - ROW0;
                bool ok = t.expert == 5 && t.rows >= 1 && t.rows <= t.height && t.height >= BM / 2 && t.height <= BM &&
                          t.height % 32 == 0 && t.nt >= 0 && t.nt < NT && first >= 0 && first + t.rows <= m_e;
                for (int r = 0; ok && r < t.rows; ++r) ++seen[t.nt][first + r];
                int rows = 0;
                for (int half = 0; ok && half < 2; ++half) {
                    const TileCoord h = tile_in_expert<BM>(5, ROW0, m_e, local, NT, half, cut);
                    if (half == 1 && t.rows <= BM / 2) {
                        ok = h.expert == kEmptySlot;
                        continue;
                    }
                    ok = h.expert == 5 && h.nt == t.nt && h.height == BM / 2 && h.row0 == t.row0 + rows && h.rows >= 1 &&
                         h.rows <= BM / 2;
                    rows += h.rows;
                }
                if (!ok || rows != t.rows) {
                    std::printf("cut %d, %d rows, tile %d\n", static_cast<int>(cut), m_e, local);
                    return -1;
                }
                ++checked;
            }
            for (int nt = 0; nt < NT; ++nt)
                for (int r = 0; r < m_e; ++r)
                    if (seen[nt][r] != 1) return -1;
        }
    return checked;
}

int main(int argc, char** argv) {
    long n = -1;
    if (argc == 3 && !std::strcmp(argv[1], "store_bounds")) n = store_bounds(std::atoi(argv[2]));
    if (argc == 2 && !std::strcmp(argv[1], "tiles")) n = tiles();
    std::printf("checked %ld\n", n);
    return n > 0 ? 0 : 1;
}
