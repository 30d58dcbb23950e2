// Test helper (CPU): reads lines "n_flat K bf16 elementwise lars" and prints
// the launch shape that the library chooses for them.
#include <cstdio>

#include "ags_internal.h"

int main() {
    long long n;
    int K, bf16, ew, lars;
    while (std::scanf("%lld %d %d %d %d", &n, &K, &bf16, &ew, &lars) == 5) {
        ags_config c{};
        c.n_flat = n;
        c.K = K;
        c.grad_dtype = bf16 ? AGS_BF16 : AGS_F32;
        c.mode = lars ? AGS_MODE_LARS : AGS_MODE_AGS;
        c.elementwise = ew;
        const ags::LaunchShape s = ags::launch_shape(c);
        std::printf("%d %d %d %d %d %d %d\n", s.step_blocks, s.stats_blocks, s.update_blocks,
                    (int)s.stream_step, (int)s.stream_update, (int)s.stream_gbar, (int)s.grouped_step);
    }
}
