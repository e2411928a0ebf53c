// The voxelizer's workspace, for any number of triangles and any 16-byte aligned start: the
// parts follow one another inside the size that the query gives, and the slot counter's
// 128-byte line holds nothing that the raster pass reads; exits 1 otherwise.
#include "emu.h"
#include "voxelize.hip"

int main() {
    int bad = 0;
    for (int n : {1, 4, 32})
        for (int surface = 0; surface < 2; ++surface)
            for (long long t = 1; t < 5000; t = t < 300 ? t + 1 : t + 97)
                for (uintptr_t start = 4096; start < 4096 + 128; start += 16) {
                    const VoxWorkspace w = vox_workspace(reinterpret_cast<void*>(start), n, t, surface != 0);
                    const uintptr_t end = start + vct_voxelize_workspace_size(n, t, surface != 0);
                    const uintptr_t line = (uintptr_t)w.counter & ~uintptr_t(127);
                    const bool in_order = (uintptr_t)(w.setup + t) <= (uintptr_t)w.offs && w.offs + t <= w.total &&
                                          (uintptr_t)(w.total + 1) <= (uintptr_t)w.counter &&
                                          (uintptr_t)(w.counter + 1) <= (uintptr_t)w.bsum &&
                                          (uintptr_t)(w.bsum + (t + kScanBlock - 1) / kScanBlock) <= end;
                    if ((!in_order || (uintptr_t)(w.total + 1) > line) && ++bad < 5)
                        printf("n %d, %lld triangles, surface %d, start %zu\n", n, t, surface, (size_t)start);
                }
    printf("%d layouts wrong\n", bad);
    return bad != 0;
}
