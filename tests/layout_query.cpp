// Prints the launch shapes that the library plans for a molecule of given sizes: host
// code only, linked against the library.  One query per line on stdin:
//   layout nao naux_pad nf_pad aux_slab k_tile tuned_tile tuned_splits nocc precision with_D delta nsplit overlap force_slab ktile
// answered by "ktile nsplit_k nsub slab nslab kdim bytes kpart_bytes", and
//   candidates nao naux_pad nf_pad aux_slab k_tile tuned_tile tuned_splits nocc precision
// by the autotuner's "tile splits" pairs, and
//   static nao naux_pad nf_pad aux_slab k_tile tuned_tile tuned_splits nocc precision
// by "fits ktile nsplit_k slab bytes" of the build in static scratch.
#include <iostream>
#include <string>

#include "dfjk_internal.h"

using namespace dfjk;

int main()
{
    std::string what;
    while (std::cin >> what) {
        Plan p;
        p.stage = 1;
        int nocc, precision;
        KShape tuned;
        std::cin >> p.nao >> p.naux_pad >> p.nf_pad >> p.aux_slab >> p.k_tile >> tuned.tile >> tuned.nsplit >> nocc >> precision;
        if (tuned.tile != 0) p.tuned[(int64_t)nocc * 8 + precision] = tuned;
        p.naux = p.naux_pad;
        p.nf = p.nf_pad;
        if (what == "layout") {
            int with_D, delta, nsplit, overlap, ktile;
            int64_t force_slab;
            std::cin >> with_D >> delta >> nsplit >> overlap >> force_slab >> ktile;
            const BuildLayout L = build_layout(p, nocc, precision, with_D, delta, nsplit, overlap, force_slab, ktile);
            const int64_t tiles = delta ? (int64_t)L.ntile * L.ntile : (int64_t)L.ntile * (L.ntile + 1) / 2;
            std::cout << L.ktile << ' ' << L.nsplit_k << ' ' << L.nsub << ' ' << L.slab << ' ' << L.nslab << ' '
                      << L.kdim << ' ' << L.bytes << ' ' << L.nslab * L.nsplit_k * tiles * L.ktile * L.ktile * 8
                      << '\n';
        } else if (what == "static") {
            BuildLayout L;
            const bool fits = static_layout(p, nocc, precision, false, L);
            std::cout << fits << ' ' << L.ktile << ' ' << L.nsplit_k << ' ' << L.slab << ' ' << L.bytes << '\n';
        } else {
            for (const KShape &c : autotune_candidates(p, nocc, precision)) std::cout << c.tile << ' ' << c.nsplit << ' ';
            std::cout << '\n';
        }
    }
}
