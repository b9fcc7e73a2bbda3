// Host test of the scratch buffer (ss_scratch.hpp) against a device with so
// much memory: what a wish beyond the need may cost, and may not.
#include <cstdio>
#include <cstdlib>
#include <map>

#include "ss_scratch.hpp"

struct FakeOps {
    int64_t memory = 1000, used = 0;  // floats
    int allocs = 0, failed = 0, frees = 0, syncs = 0, fail_sync = 0;
    bool capture = false;
    std::map<void *, int64_t> sizes;
    int dev_alloc(void **p, size_t bytes) {
        const int64_t n = (int64_t)(bytes / sizeof(float));
        if (used + n > memory) { ++failed; return 2; }
        ++allocs;
        used += n;
        *p = std::malloc(1);
        sizes[*p] = n;
        return 0;
    }
    void dev_free(void *p) {
        ++frees;
        used -= sizes[p];
        sizes.erase(p);
        std::free(p);
    }
    int device_sync() {
        ++syncs;
        if (fail_sync) { --fail_sync; return 7; }
        return 0;
    }
    bool capturing() { return capture; }
    int calls() const { return allocs + failed + frees + syncs; }
};

static int failures = 0;
#define CHECK(c)                                                    \
    do {                                                            \
        if (!(c)) {                                                 \
            std::printf("FAILED line %d: %s\n", __LINE__, #c);      \
            ++failures;                                             \
        }                                                           \
    } while (0)

int main() {
    using namespace ss;
    int code = 0;
    {   // room for the wish
        FakeOps o; ScratchBuffer s;
        CHECK(s.hold(o, 100, 200, &code) == SCRATCH_OK && s.cap == 200 && o.calls() == 1);
        CHECK(s.hold(o, 100, 200, &code) == SCRATCH_OK && o.calls() == 1);
        CHECK(s.hold(o, 150, 150, &code) == SCRATCH_OK && o.calls() == 1);
        // a larger need: the old buffer goes after the device is done with it
        CHECK(s.hold(o, 900, 900, &code) == SCRATCH_OK && s.cap == 900 && o.syncs == 1 && o.frees == 1);
        s.drop(o);
        CHECK(o.used == 0 && !s.p && s.cap == 0);
    }
    {   // no room for it: tried once, then left alone, call after call
        FakeOps o; ScratchBuffer s;
        CHECK(s.hold(o, 600, 1200, &code) == SCRATCH_OK && s.cap == 600 && o.failed == 1);
        const int before = o.calls();
        float *held = s.p;
        for (int k = 0; k < 3; ++k) CHECK(s.hold(o, 600, 1200, &code) == SCRATCH_OK && s.p == held);
        CHECK(o.calls() == before);
        // another limit: tried again, beside the buffer, which stays
        s.refused = INT64_MAX;
        CHECK(s.hold(o, 600, 1200, &code) == SCRATCH_OK && s.p == held && o.frees == 0 && o.syncs == 0);
        s.drop(o);
    }
    {   // a buffer that suffices is never given up before its successor is there
        FakeOps o; ScratchBuffer s;
        CHECK(s.hold(o, 700, 700, &code) == SCRATCH_OK);
        float *held = s.p;
        CHECK(s.hold(o, 500, 900, &code) == SCRATCH_OK && s.p == held && s.cap == 700 && o.frees == 0);
        s.drop(o);
        CHECK(s.hold(o, 300, 300, &code) == SCRATCH_OK);
        CHECK(s.hold(o, 250, 500, &code) == SCRATCH_OK && s.cap == 500 && o.used == 500);
        s.drop(o);
    }
    {   // under capture nothing is waited for, freed or allocated for a wish
        FakeOps o; ScratchBuffer s;
        CHECK(s.hold(o, 300, 300, &code) == SCRATCH_OK);
        o.capture = true;
        const int before = o.calls();
        CHECK(s.hold(o, 300, 600, &code) == SCRATCH_OK && s.cap == 300 && o.calls() == before);
        o.capture = false;
        CHECK(s.hold(o, 300, 600, &code) == SCRATCH_OK && s.cap == 600);
        s.drop(o);
    }
    {   // failures
        FakeOps o; ScratchBuffer s;
        CHECK(s.hold(o, 2000, 4000, &code) == SCRATCH_ALLOC && code == 2 && !s.p && s.cap == 0);
        CHECK(s.hold(o, 300, 300, &code) == SCRATCH_OK);
        o.fail_sync = 1;
        CHECK(s.hold(o, 400, 400, &code) == SCRATCH_SYNC && code == 7 && s.cap == 300 && s.p);
        o.fail_sync = 1;
        CHECK(s.hold(o, 300, 400, &code) == SCRATCH_SYNC && s.cap == 300 && o.used == 300);
        CHECK(s.hold(o, 400, 400, &code) == SCRATCH_OK && s.cap == 400);
        s.drop(o);
        CHECK(o.used == 0);
    }
    if (failures == 0) std::printf("all checks passed\n");
    return failures != 0;
}
