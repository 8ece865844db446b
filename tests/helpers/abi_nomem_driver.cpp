// lll_plan_nodes with no host memory to be had: the call has to return a status, since no
// exception may leave the C ABI.  Linked against the host-only launchers
// (abi_host_stubs.cpp); operator new fails while `exhausted` is set.
#include <cstdio>
#include <cstdlib>
#include <new>

#include "lll.h"
#include "lll_internal.hpp"

static bool exhausted = false;

void *operator new(std::size_t n) {
    void *p = exhausted ? nullptr : std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void *operator new(std::size_t n, const std::nothrow_t &) noexcept {
    return exhausted ? nullptr : std::malloc(n ? n : 1);
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }
void operator delete(void *p, const std::nothrow_t &) noexcept { std::free(p); }

int main() {
    lll_plan plan;
    plan.N = 40;
    plan.s = 100000;
    plan.K = plan.N * plan.s;
    int32_t count[40];
    exhausted = true;
    const int rc = lll_plan_nodes(&plan, count, nullptr, nullptr, nullptr);
    exhausted = false;
    std::printf("%d\n", rc);
    return rc == LLL_ENOMEM || rc == LLL_EHIP ? 0 : 1;
}
