// An asynchronous call whose result is first looked at when the host has no memory left for the library: an error code, and an empty
// result instead of one whose views hold bounds.  operator new of this program is the one the library calls too; only allocations
// asked for by the library itself fail.  Needs a GPU; built and run by tests/test_gpu_c_abi.py.
#include <dlfcn.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

#include "bms.h"

static long left = -1; // allocations of the library until they fail; -1: never

void *operator new(std::size_t bytes)
{
    Dl_info by;
    if (left >= 0 && dladdr(__builtin_return_address(0), &by) && by.dli_fname && std::strstr(by.dli_fname, "libbms.so") && left-- == 0) {
        left = 0;
        throw std::bad_alloc();
    }
    if (void *p = std::malloc(bytes ? bytes : 1))
        return p;
    throw std::bad_alloc();
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }

#define CHECK(x)                                                                                                       \
    do {                                                                                                               \
        if (!(x)) {                                                                                                    \
            std::printf("line %d: %s (%s)\n", __LINE__, #x, bms_last_error());                                         \
            return 1;                                                                                                  \
        }                                                                                                              \
    } while (0)

int main()
{
    const int64_t n = 2000;
    std::vector<int64_t> rowptr;
    std::vector<int32_t> col;
    for (int64_t v = 0; v <= n; ++v)
        rowptr.push_back(v * 8);
    for (int64_t v = 0; v < n; ++v)
        for (int j = 0; j < 8; ++j)
            col.push_back((int32_t)((v % 250) + 250 * j)); // ascending
    bms_csr *csr = nullptr;
    CHECK(bms_csr_load(rowptr.data(), col.data(), n, n * 8, BMS_HOST, &csr) == BMS_OK);
    std::vector<int32_t> seeds;
    for (int32_t i = 0; i < 4 * 32; ++i)
        seeds.push_back(i * 7 % n);
    const int32_t fanouts[2] = {4, 3};
    bms_result *res = nullptr;
    bms_opts opts{};
    int failed = 0;
    for (long allowed = 0;; ++allowed) {
        for (int call = 0; call < 3; ++call) { // the third one is asynchronous
            opts.flags = call == 2 ? BMS_ASYNC : 0;
            opts.recycle = res;
            CHECK(bms_sample_nodewise(csr, seeds.data(), 4, 32, fanouts, 2, 5, &opts, &res) == BMS_OK);
        }
        while (bms_result_ready(res) == 0)
            ;
        left = allowed;
        const int rc = bms_result_wait(res);
        const bool all = left >= 0 && rc == BMS_OK;
        left = -1;
        bms_hop_view view;
        if (all) {
            CHECK(bms_result_hop(res, 1, &view) == BMS_OK && view.nnz > 0 && view.nnz <= 3 * view.rows && view.ncols > 0);
            break;
        }
        ++failed;
        CHECK(rc == BMS_ENOMEM);
        int32_t k = -1, L = -1;
        CHECK(bms_result_info(res, &k, &L) == BMS_OK && k == 0 && L == 0);
        CHECK(bms_result_hop(res, 1, &view) == BMS_EINVAL && bms_result_wait(res) == BMS_OK);
        CHECK(allowed < 100);
    }
    CHECK(failed > 0);
    std::printf("%d failures, each an error and an empty result\n", failed);
    bms_free(res);
    bms_free(csr);
    return 0;
}
