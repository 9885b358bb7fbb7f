// Answers questions about the library's routing rules (csrc/routes.hpp) for
// the tests: one question per line of standard input, one answer per line.
//   march LATTICE BYTES NX NY NZ BCX BCY BCZ MASK COMP CUS
//     planes per segment of the two-step launches, -1: one-step launches
#include <iostream>
#include <string>

#include "../paper_2201_11330_amd/csrc/routes.hpp"

using namespace imexlbm;

int main()
{
    std::string what;
    while (std::cin >> what) {
        if (what != "march") return 1;
        MarchBox b;
        int cus = 0;
        std::cin >> b.lattice >> b.storage_bytes >> b.n[0] >> b.n[1] >> b.n[2] >> b.bc[0] >> b.bc[1] >> b.bc[2] >>
            b.mask >> b.comp >> cus;
        std::cout << march_route(b, cus) << "\n";
    }
    return 0;
}
