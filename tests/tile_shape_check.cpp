// CPU build of the NUFFT tile-shape rule (paper_2603_17166_amd/csrc/nufft_index.h):
// prints the shape for "rows columns W points" on the command line.
#include <cstdio>
#include <cstdlib>

#include "nufft_index.h"

int main(int argc, char **argv) {
    if (argc != 5) return 2;
    int tx = 0, ty = 0;
    psht::tile_shape(std::atoi(argv[1]), std::atoi(argv[2]), std::atoi(argv[3]), std::atoll(argv[4]), tx, ty);
    std::printf("%dx%d\n", tx, ty);
    return 0;
}
