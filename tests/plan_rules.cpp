// Prints how launches of two steps would go (two_step_plan) on a device of 256
// compute units, and the first case's default tile of single steps.  One launch
// per line of input: alone (0/1), precision (LBM_AXI_*), collision form
// (COLLIDE_*), the number of cases, then nr, nz, z_periodic of each.
#include "../paper_1810_09299_amd/csrc/case_internal.hpp"

#include <cstdio>
#include <vector>

int main()
{
    int alone, precision, mode, n;
    while (scanf("%d %d %d %d", &alone, &precision, &mode, &n) == 4) {
        std::vector<lbm_axi_case> cases(n);
        std::vector<const lbm_axi_case *> ptrs;
        for (lbm_axi_case &c : cases) {
            if (scanf("%d %d %d", &c.prm.nr, &c.prm.nz, &c.prm.z_periodic) != 3) return 1;
            c.prm.precision = precision;
            c.P64.mode = c.P32.mode = mode;
            c.cus = 256;
            ptrs.push_back(&c);
        }
        const axi::TwoStepPlan p = axi::two_step_plan(ptrs.data(), n, alone != 0);
        // tile -1: singly (a batch of one collision form decides as build_pairs does)
        const bool singly = !p.march && (p.tile < 0 || (!alone && axi::singly_ahead(p.single_us, p.pairs_us)));
        printf("%d %d %d %d %d\n", (int)p.march, p.waves, p.rows, singly ? -1 : p.tile, axi::default_tile(ptrs[0]));
    }
    return 0;
}
