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

int main(int argc, char** argv) {
    long n = -1;
    if (argc == 3 && !std::strcmp(argv[1], "store_bounds")) n = store_bounds(std::atoi(argv[2]));
    std::printf("checked %ld\n", n);
    return n > 0 ? 0 : 1;
}
