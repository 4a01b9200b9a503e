// The pool of device memory (csrc/device_pool.hpp) over a stand-in for the runtime: what is handed out, kept and given
// back, and that nothing is lost while the runtime refuses to allocate and free, as it does while a thread captures.
// Built and run by tests/test_planner_sanitizers.py.
#include <cstdio>
#include <cstdlib>
#include <map>
#include "device_pool.hpp"
using smha::DevicePool;
static std::map<void *, size_t> live;
static size_t in_use = 0, capacity = (size_t)64 << 20;
static bool capturing = false;
static int allocate(void **ptr, size_t bytes) {
    if (capturing || in_use + bytes > capacity) return 1;
    *ptr = std::malloc(1);
    live[*ptr] = bytes;
    in_use += bytes;
    return 0;
}
static int release(void *ptr) {
    if (capturing) return 1;
    const auto it = live.find(ptr);
    if (it == live.end()) std::abort();  // (not allocated, or given back twice)
    in_use -= it->second;
    live.erase(it);
    std::free(ptr);
    return 0;
}
static void expect(bool ok, const char *what) {
    if (ok) return;
    printf("failed: %s\n", what);
    std::exit(1);
}
int main() {
    DevicePool pool(allocate, release);
    void *a = nullptr, *b = nullptr, *c = nullptr;
    expect(pool.take(&a, 100, 0) == 0 && live[a] == 64 << 10, "at least 64 KB");
    pool.give(a, 100, 0, true);
    expect(live.count(a) == 1, "an idle block is kept");
    expect(pool.take(&b, 65536, 1) == 0 && b != a, "another device's block is not handed out");
    expect(pool.take(&c, 65537, 0) == 0 && c != a && live[c] == 128 << 10, "nor one that is too small");
    pool.give(c, 65537, 0, false);
    expect(live.count(c) == 0, "a block that is not idle goes back");
    capturing = true;
    expect(pool.take(&c, 1 << 20, 0) != 0, "a capture refuses a new block");
    expect(pool.take(&c, 7, 0) == 0 && c == a, "what was kept is still there after that refusal");
    pool.give(c, 7, 0, true);
    capturing = false;
    expect(pool.take(&c, 7, 0) == 0 && c == a, "and after it was given back during the capture");
    pool.give(c, 7, 0, true);
    pool.give(b, 65536, 1, true);
    expect(in_use == 128 << 10, "two blocks kept");
    void *big = nullptr;
    expect(pool.take(&big, (1 << 20) + 1, 0) == 0 && live[big] == (1 << 20) + 1, "no rounding above 1 MB");
    pool.give(big, (1 << 20) + 1, 0, true);
    expect(live.count(big) == 0, "above 1 MB nothing is kept");
    void *many[40];
    for (void *&p : many) expect(pool.take(&p, 1 << 20, 0) == 0, "40 blocks");
    for (void *p : many) pool.give(p, 1 << 20, 0, true);
    expect(in_use <= DevicePool::kAtMost && in_use > DevicePool::kAtMost - (1 << 20), "16 MB kept at most");
    expect(pool.fresh(&big, capacity) == 0 && in_use == capacity, "what is kept goes back when there is no memory");
    release(big);
    expect(in_use == 0 && live.empty(), "nothing is lost");
    printf("device pool ok\n");
    return 0;
}
