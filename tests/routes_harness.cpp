// Answers questions about the library's routing rules (csrc/routes.hpp) for
// the tests: one question per line of standard input, one answer per line.
//   march LATTICE BYTES NX NY NZ BCX BCY BCZ MASK COMP CUS
//     planes per segment of the two-step launches, -1: one-step launches
//   2d NX NY STORAGE WALLS MASK COMP STEPS
//     steps per launch of strips, regions, most and fewest steps per launch,
//     then the launches that make STEPS steps, each as steps and regions
//     (regions -1: strips; steps 1: a one-step launch)
#include <iostream>
#include <string>

#include "../paper_2201_11330_amd/csrc/routes.hpp"

using namespace imexlbm;

int main()
{
    std::string what;
    while (std::cin >> what) {
        if (what == "2d") {
            Box2D b;
            int steps = 0;
            std::cin >> b.nx >> b.ny >> b.storage >> b.walls >> b.mask >> b.comp >> steps;
            const Route2D r = route_2d(b);
            std::cout << r.strips << " " << r.regions << " " << r.most << " " << r.fewest;
            while (steps > 0) {
                const int k = next_launch(r, steps);
                if (k > 0) std::cout << " " << k << " " << (k == r.strips ? -1 : int(launch_regions(r, k)));
                else std::cout << " 1 -1";
                steps -= k > 0 ? k : 1;
            }
            std::cout << "\n";
            continue;
        }
        if (what != "march") return 1;
        MarchBox b;
        int cus = 0;
        std::cin >> b.lattice >> b.storage_bytes >> b.n[0] >> b.n[1] >> b.n[2] >> b.bc[0] >> b.bc[1] >> b.bc[2] >>
            b.mask >> b.comp >> cus;
        std::cout << march_route(b, cus) << "\n";
    }
    return 0;
}
