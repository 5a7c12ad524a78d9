// adjoint_room_driver.cpp -- test-only: kt_adjoint with workspaces of the least
// size and of more, linked with the host stand-ins of the kernel launchers
// (stub_launch.cpp), which touch all the memory that the kernels would.  Every
// workspace ends at the end of its allocation, so that a store that reaches past
// the bytes given is an AddressSanitizer report.
#include <cstdint>
#include <cstdio>
#include <cstdlib>

#include "kerrtrace.h"

int main() {
    const int dims[][2] = {{1, 1}, {33, 31}, {301, 300}};
    const size_t more[] = {0, 1, 47, 48, 4096, 1000003};
    int calls = 0;
    for (auto& d : dims)
        for (int every : {0, 1, 1024})
            for (int split : {-1, 0, 300})
                for (size_t extra : more) {
                    const kt_camera cam = {1000.0, 0.8, 35.0, 35.0, d[0], d[1]};
                    const kt_spacetime st = {1.0, 0.7, KT_METRIC_KERR, 0.0};
                    const kt_disk disk = {1, 3.4, 30.0, 2.0, KT_ROT_KEPLER, 0.0, KT_EMIS_TAPERED};
                    kt_integrator it = {};
                    it.method = KT_DP45;
                    it.precision = KT_FP64;
                    it.rtol = it.atol = 1e-12;
                    it.h_init = 1.0;
                    it.capture_buffer = 0.01;
                    it.max_steps = 300;
                    it.checkpoint_every = every;
                    it.split_above = split;
                    const size_t n = static_cast<size_t>(d[0]) * d[1];
                    const size_t bytes = kt_adjoint_workspace_bytes(&cam, &it) + extra;
                    // the end of the buffer is its last byte; the start is aligned
                    void* ws = nullptr;
                    if (posix_memalign(&ws, 256, bytes)) return 2;
                    auto* fate = static_cast<uint8_t*>(std::malloc(n));
                    auto* cot = static_cast<double*>(std::malloc(8 * n));
                    auto* steps = static_cast<int32_t*>(std::malloc(4 * n));
                    const int rc = kt_adjoint(&cam, &st, &disk, &it, fate, nullptr, steps, cot, nullptr, nullptr, nullptr,
                                              nullptr, nullptr, ws, bytes, nullptr);
                    if (rc != KT_OK) {
                        std::printf("rc %d: %s\n", rc, kt_last_error());
                        return 1;
                    }
                    ++calls;
                    std::free(ws);
                    std::free(fate);
                    std::free(cot);
                    std::free(steps);
                }
    std::printf("ok %d\n", calls);
    return 0;
}
