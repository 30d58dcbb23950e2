// Test program: the largest size operator new is asked for within a call of
// ags_stats_noalloc on 12,000 layers.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <new>
#include <vector>

#include "ags.h"

static std::size_t largest;
void* operator new(std::size_t n) {
    if (n > largest) largest = n;
    if (void* p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

int main() {
    const int L = 12000, K = 2, each = 8, pad = AGS_ALIGN_ELEMS;
    std::vector<ags_layer> layers(L);
    for (int l = 0; l < L; ++l) {
        layers[l] = ags_layer{};
        layers[l].offset = (int64_t)l * pad;
        layers[l].numel = each;
    }
    ags_config c{};
    c.n_layers = L;
    c.layers = layers.data();
    c.n_flat = (int64_t)L * pad;
    c.K = K;
    c.grad_dtype = AGS_F32;
    c.mode = AGS_MODE_AGS;
    c.lr = 0.1;
    c.delta = 0.5;
    float *w = nullptr, *g = nullptr;
    const size_t bytes = (size_t)c.n_flat * sizeof(float);
    if (hipMalloc(reinterpret_cast<void**>(&w), bytes) != hipSuccess ||
        hipMalloc(reinterpret_cast<void**>(&g), K * bytes) != hipSuccess ||
        hipMemset(w, 0, bytes) != hipSuccess || hipMemset(g, 0, K * bytes) != hipSuccess)
        return 2;
    std::vector<ags_layer_stats> out(L);
    ags_global_stats glob{};
    for (int i = 0; i < 2; ++i) {  // the first call loads the kernels
        largest = 0;
        const ags_status s = ags_stats_noalloc(&c, w, g, c.n_flat, out.data(), &glob, nullptr);
        if (s != AGS_OK) {
            std::fprintf(stderr, "%s: %s\n", ags_status_string(s), ags_last_error(nullptr));
            return 1;
        }
    }
    std::printf("%zu\n", largest);
    return hipFree(w) == hipSuccess && hipFree(g) == hipSuccess ? 0 : 2;
}
