// ss_scratch.hpp -- a context's device scratch, grown on demand.
//
// Written against a small set of device operations (`Ops`) so that it
// compiles without HIP, as ss_geom_upload.hpp is; the integers are 0 on
// success and an error code otherwise:
//
//   int dev_alloc(void **p, size_t bytes);   // leaves no pending error behind
//   void dev_free(void *p);
//   int device_sync();    // all enqueued work done (the old buffer unused)
//   bool capturing();     // the call's stream is being captured
#pragma once

#include <cstddef>
#include <cstdint>

namespace ss {

enum ScratchError { SCRATCH_OK = 0, SCRATCH_SYNC, SCRATCH_ALLOC };

struct ScratchBuffer {
    float *p = nullptr;
    int64_t cap = 0;              // floats
    int64_t refused = INT64_MAX;  // smallest `want` beyond a `need` that found no memory

    // Hold at least `need` floats, and `want` >= need where there is room: a
    // buffer that already holds `need` is given up only for a larger one that
    // is there, never while the stream is captured, and a size that found no
    // memory is not tried again while `refused` stands.  On failure `*code`
    // receives the operation's error code.
    template <class Ops>
    ScratchError hold(Ops &ops, int64_t need, int64_t want, int *code) {
        if (want <= cap) return SCRATCH_OK;
        const bool enough = need <= cap;
        if (enough && (want >= refused || ops.capturing())) return SCRATCH_OK;
        int e;
        if (!enough && p) {
            // too small in any case; enqueued work may still use it
            if ((e = ops.device_sync()) != 0) { *code = e; return SCRATCH_SYNC; }
            drop(ops);
        }
        if (want > need && want < refused) {
            void *q = nullptr;
            if (ops.dev_alloc(&q, (size_t)want * sizeof(float)) == 0) {
                if (p) {
                    if ((e = ops.device_sync()) != 0) {
                        ops.dev_free(q);
                        *code = e;
                        return SCRATCH_SYNC;
                    }
                    drop(ops);
                }
                p = static_cast<float *>(q);
                cap = want;
                return SCRATCH_OK;
            }
            refused = want;
        }
        if (enough) return SCRATCH_OK;
        void *q = nullptr;
        if ((e = ops.dev_alloc(&q, (size_t)need * sizeof(float))) != 0) { *code = e; return SCRATCH_ALLOC; }
        p = static_cast<float *>(q);
        cap = need;
        return SCRATCH_OK;
    }

    // (enqueued work must be done with it)
    template <class Ops>
    void drop(Ops &ops) {
        if (p) ops.dev_free(p);
        p = nullptr;
        cap = 0;
    }
};

}  // namespace ss
