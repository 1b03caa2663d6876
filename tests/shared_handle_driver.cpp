// CPU-only test driver: threads that drive a GPU each share a neighbourhood in the allocation-free call, whose handle
// builds every schedule in the first call that asks for it.  Run under ThreadSanitizer against the stand-in HIP runtime of
// hip_stub_runtime.cpp; ends with "shared handle ok".
#include <atomic>
#include <cstdio>
#include <thread>
#include <vector>

#include "iso.h"

extern "C" {
void *stub_device_alloc(size_t bytes);
void stub_device_free(void *q);
long stub_kernel_launches(void);
}

int main() {
    const int32_t dims[2] = {9, 7}, offs[] = {0, 1, 1, 0, -1, 2, 3, 3, 0, 0};
    const int s = 5, threads = 4;
    const size_t bytes = 63 * (size_t)s * 40;
    for (int turn = 0; turn < 20; ++turn) {
        iso_comm_t comm = nullptr;
        if (iso_neighborhood_create(2, dims, s, offs, &comm) != ISO_SUCCESS) return 1;
        std::atomic<int> bad{0}, ready{0};
        std::vector<std::thread> all;
        for (int t = 0; t < threads; ++t)
            all.emplace_back([&, t] {
                void *send = stub_device_alloc(bytes), *recv = stub_device_alloc(bytes);
                ++ready;
                while (ready < threads) std::this_thread::yield();
                for (int q = 0; q <= ISO_ALG_COMBINED_STAGED; ++q) {
                    const int alg = turn & 1 ? q : (q + t) % (ISO_ALG_COMBINED_STAGED + 1);
                    if (iso_neighbor_alltoall_noalloc(send, recv, 40, comm, alg, nullptr) != ISO_SUCCESS) ++bad;
                }
                if (iso_neighbor_alltoall_noalloc(send, recv, 40, comm, 77, nullptr) != ISO_ERR_ARG) ++bad;
                stub_device_free(send);
                stub_device_free(recv);
            });
        for (std::thread &t : all) t.join();
        if (bad || iso_neighborhood_free(&comm) != ISO_SUCCESS) return 2;
    }
    if (stub_kernel_launches() < 20 * threads * 6) return 3;
    std::printf("shared handle ok\n");
    return 0;
}
