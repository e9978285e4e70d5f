// bq_step_plan_create when the host's memory runs out: every allocation it makes
// fails in turn, and each time it must report an error, return no plan and leave
// nothing allocated.  The program replaces operator new and the first HIP call a
// plan makes (no GPU is used); run by tests/test_plan_alloc_failure.py.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <vector>

#include "bq.h"

namespace {
bool counting = false;
long live = 0;       // allocations made while counting and not freed
long left = -1;      // allocations until the failing one; -1: none fails
bool failed = false;

void *allocate(std::size_t n)
{
    if (counting && left >= 0 && left-- == 0) {
        failed = true;
        return nullptr;
    }
    void *p = std::malloc(n ? n : 1);
    if (p && counting)
        ++live;
    return p;
}

void release(void *p)
{
    if (p && counting)
        --live;
    std::free(p);
}

void *or_throw(void *p)
{
    if (!p)
        throw std::bad_alloc();
    return p;
}
}  // namespace

void *operator new(std::size_t n) { return or_throw(allocate(n)); }
void *operator new[](std::size_t n) { return or_throw(allocate(n)); }
void *operator new(std::size_t n, const std::nothrow_t &) noexcept { return allocate(n); }
void *operator new[](std::size_t n, const std::nothrow_t &) noexcept { return allocate(n); }
void operator delete(void *p) noexcept { release(p); }
void operator delete[](void *p) noexcept { release(p); }
void operator delete(void *p, std::size_t) noexcept { release(p); }
void operator delete[](void *p, std::size_t) noexcept { release(p); }

extern "C" hipError_t hipGetDevice(int *) { return hipErrorNoDevice; }

int main()
{
    // descriptors only: nothing is read through the pointers
    std::vector<bq_tensor> list(50);
    for (std::size_t i = 0; i < list.size(); ++i) {
        bq_tensor &t = list[i];
        char *at = reinterpret_cast<char *>(static_cast<uintptr_t>(4096 * (i + 1)));
        t.param = reinterpret_cast<float *>(at);
        t.grad = at;
        t.state1 = t.state2 = reinterpret_cast<uint8_t *>(at);
        t.absmax1 = t.absmax2 = reinterpret_cast<float *>(at);
        t.numel = 100 + 5000 * static_cast<int64_t>(i);
    }
    int bad = 0;
    for (const bq_optimizer opt : {BQ_ADAM, BQ_LAMB}) {
        for (const int big : {0, 1}) {  // records made on the host, on the device
            list.back().numel = big ? int64_t{1} << 27 : 100;
            int made = 0;
            for (;; ++made) {
                bq_step_plan plan = reinterpret_cast<bq_step_plan>(&bad);
                live = 0;
                left = made;
                failed = false;
                counting = true;
                const bq_status s = bq_step_plan_create(opt, 2048, BQ_F32, list.data(),
                                                        static_cast<int32_t>(list.size()), &plan);
                counting = false;
                if (s != BQ_ERR_HIP || plan != nullptr || live != 0) {
                    std::printf("optimizer %d, list %d, allocation %d: status %d, plan %p, "
                                "%ld left\n", (int)opt, big, made, (int)s, (void *)plan, live);
                    bad = 1;
                }
                if (!failed)
                    break;  // all allocations succeeded; the HIP call failed
            }
            std::printf("optimizer %d, list %d: %d allocations\n", (int)opt, big, made);
            if (made < 3)
                bad = 1;  // operator new was not replaced for the library
        }
    }
    std::puts(bad ? "plan_alloc_failure FAILED" : "plan_alloc_failure ok");
    return bad;
}
