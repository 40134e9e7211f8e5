// Entry points of the library when the host has no memory left: an error code, not an exception through C.  operator new of this
// program is the one the library calls too.  Needs no GPU: the handle is allocated before the first device call.
// Built and run by tests/test_abi.py.
#include <cstdio>
#include <cstdlib>
#include <new>

#include "bms.h"

static long left = -1; // allocations until they fail; -1: never

void *operator new(std::size_t bytes)
{
    if (left == 0)
        throw std::bad_alloc();
    if (left > 0)
        --left;
    if (void *p = std::malloc(bytes ? bytes : 1))
        return p;
    throw std::bad_alloc();
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }

int main()
{
    const int64_t rowptr[3] = {0, 1, 2};
    const int32_t col[2] = {1, 0};
    bms_csr *csr = nullptr;
    for (long allowed = 0; allowed < 4; ++allowed) {
        left = allowed;
        const int rc = bms_csr_load(rowptr, col, 2, 2, BMS_HOST, &csr);
        left = -1;
        std::printf("%ld allocations: %d %s\n", allowed, rc, bms_last_error());
        if (rc != BMS_ENOMEM || csr)
            return 1;
    }
    return 0;
}
