// Reads requests from stdin, one a line, and answers from the library's launch
// rules (host code only; nothing is launched):
//   chunks <columns> <nz> <slots>   -> the number of chunks of a marching kernel
//   tried <columns> <nz> <slots>    -> the same by trying every count
#include <cstdio>
#include <cstring>

#include "../../paper_1405_6162_amd/csrc/launch.h"

static int tried(int64_t columns, int nz, int slots) {
    int64_t best = INT64_MAX;
    int chunks = 1;
    for (int64_t c = (nz + 127) / 128; c <= nz; ++c) {
        const int64_t cost = (columns * c + slots - 1) / slots * ((nz + c - 1) / c + 3);
        if (cost < best) { best = cost; chunks = (int)c; }
    }
    return chunks;
}

int main() {
    char what[32];
    long long a, b, c;
    while (std::scanf("%31s %lld %lld %lld", what, &a, &b, &c) == 4) {
        if (!std::strcmp(what, "chunks")) std::printf("%d\n", lbl::chunks_of(a, (int)b, (int)c));
        else if (!std::strcmp(what, "tried")) std::printf("%d\n", tried(a, (int)b, (int)c));
        else return 1;
    }
    return 0;
}
