// Host check of the buffers of a batch query that nb workgroups run: the first
// of them may find no helper and run any level alone, so its tables hold
// FUSED_MAX_ROWS rows and its result every slot of a level, whatever nb is
// (two or three on a device or partition of few CUs).  Exit status 0 when
// every size holds.
#include <cstdio>

#include "fused.h"

using namespace gsi;

int main() {
    int bad = 0;
    for (uint32_t nb = 2; nb <= CL_MAX_WG; nb++) {
        const uint32_t rows = cluster_table_rows(nb), out = cluster_result_rows(nb);
        if (rows < FUSED_MAX_ROWS || rows < nb * (CL_CAP_ROWS / CL_MAX_WG) || rows > CL_CAP_ROWS) bad++;
        if (out < FUSED_MAX_SLOTS || out < nb * (CL_CAP_OUT / CL_MAX_WG) || out > CL_CAP_OUT) bad++;
    }
    if (cluster_table_rows(CL_MAX_WG) != CL_CAP_ROWS || cluster_result_rows(CL_MAX_WG) != CL_CAP_OUT) bad++;
    std::printf("too small %d\n", bad);
    return bad ? 1 : 0;
}
