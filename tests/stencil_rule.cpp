// The stencil's choice of form and its launch geometry, from the library's own
// header: for each line "epilogue gamma5-in fp64 Lx Ly Lz Lt nrhs" prints
// "split" or "chunk", the groups of right-hand sides and the number of blocks.
#include <cstdio>

#include "kernels.h"

using namespace msb;

template <typename T, int EPI, bool G5>
static void print(Geom g, int nrhs) {
    DslashArgs<T> a;
    a.g = g;
    const long nch = (g.V + CHUNK - 1) / CHUNK;
    const bool split = dslash_use_split<T, EPI, G5>(nch, nrhs);
    const long blocks = split ? dslash_split_prepare(a, nrhs) : dslash_chunk_prepare<T, G5>(a, nrhs);
    std::printf("%s %d %ld\n", split ? "split" : "chunk", split ? nrhs : (nrhs + a.rpb - 1) / a.rpb, blocks);
}
template <typename T>
static void print(int epi, int g5, Geom g, int nrhs) {
    if (g5) print<T, EPI_PLAIN, true>(g, nrhs);
    else if (epi == EPI_MV) print<T, EPI_MV, false>(g, nrhs);
    else if (epi == EPI_MV_Y) print<T, EPI_MV_Y, false>(g, nrhs);
    else if (epi == EPI_MVV) print<T, EPI_MVV, false>(g, nrhs);
    else print<T, EPI_PLAIN, false>(g, nrhs);
}

int main() {
    int epi, g5, fp64, nrhs;
    Geom g;
    while (std::scanf("%d %d %d %d %d %d %d %d", &epi, &g5, &fp64, &g.Lx, &g.Ly, &g.Lz, &g.Lt, &nrhs) == 8) {
        g.V = g.Lx * g.Ly * g.Lz * g.Lt;
        if (fp64) print<double>(epi, g5, g, nrhs);
        else print<float>(epi, g5, g, nrhs);
    }
}
