// Rules by which a launch's sizes select its kernel (csrc/lds_plan.h), over their whole range.  Exit status 0 = all hold.
#include <cstdio>
#include <initializer_list>

#include "../paper_2509_22622_amd/csrc/lds_plan.h"

// Rows of one head a CU has time for while the busiest CU works, as a share of what 256 evenly loaded CUs would take: the
// workgroups of the resident-key kernel, one per CU, each with 1 / parts of a head's rows.
static double share_at_work(int heads) {
    const int parts = heads < 256 ? 256 / heads : 1, workgroups = heads * parts;
    return double(workgroups) / double((workgroups + 255) / 256 * 256);
}

int main() {
    for (int heads = 1; heads <= 1024; ++heads)
        for (int rows : {1, 300, 512, 513, 1170, 4680, 100000}) {
            const bool taken = ll::resident_fills_chip(heads, rows, 8);
            if (!ll::resident_fills_chip(heads, rows, 2)) {
                std::printf("%d heads x %d rows: two kblocks are faster resident\n", heads, rows);
                return 1;
            }
            if (taken && rows > 512 && share_at_work(heads) < 0.66) {
                std::printf("%d heads x %d rows: the resident kernel would keep %.2f of the CUs at work\n", heads, rows, share_at_work(heads));
                return 1;
            }
            if (!taken && share_at_work(heads) >= 0.75) {
                std::printf("%d heads x %d rows: the resident kernel would fill the chip\n", heads, rows);
                return 1;
            }
        }
    std::printf("launch rules ok\n");
    return 0;
}
