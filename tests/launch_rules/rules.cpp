// Prints the launch rules' choices for the launches on stdin (built for the
// host alone by tests/test_launch_rules.py; no kernel is instantiated).
//   tile FAMILY DTYPE Lx Ly Lz NB EPILOGUE   ->   elements per lane, lanes
//   walk FAMILY DTYPE Lx Ly Lz NB GROUPS     ->   planes per walk, 1 along y
//                                                 (short tile, workgroups per XCD)
//   adjoint FAMILY DTYPE Lx Ly Lz NB KERNEL ELEMS -> 0 direct, 1 staged with the
//                                                 run-time epilogue, 2 with its own
//   batch NORB DTYPE NB LENGTHS... 0              -> 1 staged, 1 the longer tile
//                                                 (cubes of the lengths)
//   rotate DTYPE ROWS NX NY ACCUMULATE            -> 1 one thread per entry
#include <cstdio>
#include <cstring>
#include <string>

#include "pv_sweep.hpp"

namespace {

template <class P>
pv::StagedTile tile(const pv::SweepParams& p) {
    return p.dtype == 0 ? pv::staged_tile<P, double>(p, 256) : pv::staged_tile<P, float>(p, 256);
}

template <class P>
pv::StagedWalk walk(const pv::SweepParams& p, int G8) {
    const int TW = p.dtype == 0 ? 256 : 512, rowel = int(p.L[0]) * P::NO * p.nb;
    return pv::staged_walk<P>(p, (rowel + TW - 1) / TW, G8, false);
}

template <class P>
int adjoint(const pv::SweepParams& p) {
    return int(p.dtype == 0 ? pv::sweep_route<P, double>(p) : pv::sweep_route<P, float>(p));
}

}  // namespace

int main() {
    char what[16], name[32], ep[16];
    while (std::scanf("%15s %31s", what, name) == 2) {
        if (std::strcmp(what, "tile") == 0) {
            pv::SweepParams p{};
            long L[3];
            if (std::scanf("%d %ld %ld %ld %d %15s", &p.dtype, &L[0], &L[1], &L[2], &p.nb, ep) != 6) return 1;
            for (int k = 0; k < 3; ++k) p.L[k] = L[k];
            const std::string e = ep, n = name;
            p.ep = e == "step" ? pv::EP_STORE_Y | pv::EP_MOMENTS : (e == "plain" ? unsigned(pv::EP_STORE_Y) : unsigned(pv::EP_SERIES));
            pv::StagedTile t{};
            if (n == "ti") t = tile<pv::PatTI>(p);
            else if (n == "weyl") t = tile<pv::PatWeyl>(p);
            else if (n == "graphene4") t = tile<pv::PatGraphene4>(p);
            else return 1;
            std::printf("%d %d\n", t.e, t.nt);
        } else if (std::strcmp(what, "walk") == 0) {
            pv::SweepParams p{};
            long L[3];
            int G8;
            if (std::scanf("%d %ld %ld %ld %d %d", &p.dtype, &L[0], &L[1], &L[2], &p.nb, &G8) != 6) return 1;
            for (int k = 0; k < 3; ++k) p.L[k] = L[k];
            const std::string n = name;
            const pv::StagedWalk w = n == "ti" ? walk<pv::PatTI>(p, G8) : walk<pv::PatWeyl>(p, G8);
            std::printf("%d %d\n", w.C, w.along_y);
        } else if (std::strcmp(what, "adjoint") == 0) {
            pv::SweepParams p{};
            long L[3];
            if (std::scanf("%d %ld %ld %ld %d %d %d", &p.dtype, &L[0], &L[1], &L[2], &p.nb, &p.kernel, &p.st_E) != 7) return 1;
            for (int k = 0; k < 3; ++k) p.L[k] = L[k];
            p.ep = pv::EP_ADJOINT;
            p.z = p.gw[0] = p.gw[1] = p.gw[2] = reinterpret_cast<const void*>(uintptr_t(4096));
            const std::string n = name;
            p.n_orb = n == "ti" || n == "graphene4" ? 4 : 2;
            std::printf("%d\n", n == "ti" ? adjoint<pv::PatTI>(p)
                              : n == "weyl" ? adjoint<pv::PatWeyl>(p)
                              : n == "graphene4" ? adjoint<pv::PatGraphene4>(p) : adjoint<pv::PatGraphene2>(p));
        } else if (std::strcmp(what, "rotate") == 0) {
            long rows;
            int nx, ny, acc;
            if (std::scanf("%ld %d %d %d", &rows, &nx, &ny, &acc) != 4) return 1;
            std::printf("%d\n", int(pv::rotate_by_entry(std::stoi(name), rows, nx, ny, acc != 0)));
        } else if (std::strcmp(what, "batch") == 0) {
            const int no = std::stoi(name);
            int dtype, nb;
            long L;
            std::vector<pv::BatchRows> rows;
            if (std::scanf("%d %d", &dtype, &nb) != 2) return 1;
            while (std::scanf("%ld", &L) == 1 && L) rows.push_back({L * no * nb, (L + 7) / 8, L, L * L * L * no * nb});
            std::printf("%d %d\n", int(pv::batch_stages(rows, dtype == 0)), int(pv::batch_long_tile(rows, dtype == 0)));
        } else {
            return 1;
        }
    }
    return 0;
}
