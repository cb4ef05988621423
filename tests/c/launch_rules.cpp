// Reads requests from stdin, one a line, and answers from the library's launch
// rules (host code only; nothing is launched):
//   chunks <columns> <nz> <slots>   -> the number of chunks of a marching kernel
//   tried <columns> <nz> <slots>    -> the same by trying every count
//   march <lattice>                 -> whether LB_STEP_AUTO marches (1) or takes the two-pass step (0)
//   pair <lattice>                  -> whether single-fluid steps run two to a launch
//   layout <model> <lattice>        -> blocked, wide, wide_plane of lbl::Layout
// with <lattice> = <storage> <collision> <vvl> <nx> <ny> <nz>, numbers of lb.h.
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

// A context of the lattice read from stdin, with no workspace.
static bool read_lattice(int model, lb_ctx& c) {
    lb_params p{};
    if (std::scanf("%d %d %d %d %d %d", &p.storage, &p.collision, &p.vvl, &p.nx, &p.ny, &p.nz) != 6) return false;
    p.model = model;
    p.tau_f = p.tau_minus = p.tau_bulk = p.tau_ghost_even = p.tau_ghost_odd = 1.0;
    p.mobility = p.gamma = 1.0;
    if (lbl::check_params(&p) != LB_OK) return false;
    c.p = p;
    c.L = lbl::layout_of(&p);
    return true;
}

int main() {
    char what[32];
    while (std::scanf("%31s", what) == 1) {
        long long a, b, s;
        if (!std::strcmp(what, "chunks") || !std::strcmp(what, "tried")) {
            if (std::scanf("%lld %lld %lld", &a, &b, &s) != 3) return 1;
            std::printf("%d\n", *what == 'c' ? lbl::chunks_of(a, (int)b, (int)s) : tried(a, (int)b, (int)s));
        } else if (!std::strcmp(what, "march")) {
            lb_ctx c{};
            if (!read_lattice(LB_BINARY, c)) return 1;
            std::printf("%d\n", c.p.storage == LB_F64 ? lbl::march_pays<double>(&c)
                                : c.p.storage == LB_F32 ? lbl::march_pays<float>(&c) : lbl::march_pays<_Float16>(&c));
        } else if (!std::strcmp(what, "pair")) {
            lb_ctx c{};
            if (!read_lattice(LB_SINGLE, c)) return 1;
            std::printf("%d\n", c.p.storage == LB_F64 ? lbl::pair_pays<double>(&c)
                                : c.p.storage == LB_F32 ? lbl::pair_pays<float>(&c) : lbl::pair_pays<_Float16>(&c));
        } else if (!std::strcmp(what, "layout")) {
            lb_ctx c{};
            int model;
            if (std::scanf("%d", &model) != 1 || !read_lattice(model, c)) return 1;
            std::printf("%d %d %d\n", c.L.blocked, c.L.wide, c.L.wide_plane);
        } else {
            return 1;
        }
    }
    return 0;
}
