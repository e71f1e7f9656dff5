// The library's pinned slots (host_slots.hpp) with the five runtime calls they make replaced by stand-ins: no GPU, no
// HIP library. Ends with status 0, or prints the check that failed and ends with status 1.
#include <stdio.h>
#include <stdlib.h>

#include "host_slots.hpp"

using namespace megs;

static int g_syncs, g_mallocs;
static hipError_t g_sync = hipSuccess, g_malloc = hipSuccess, g_capturing = hipSuccess;
static hipStreamCaptureStatus g_status = hipStreamCaptureStatusNone;
static hipStreamCaptureMode g_mode = hipStreamCaptureModeGlobal, g_mode_at_malloc;

extern "C" {
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned int) {
    ++g_mallocs;
    g_mode_at_malloc = g_mode;
    if (g_malloc == hipSuccess) *p = calloc(1, bytes);
    return g_malloc;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
    *s = g_status;
    return g_capturing;
}
hipError_t hipStreamSynchronize(hipStream_t) {
    ++g_syncs;
    return g_sync;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) {
    const hipStreamCaptureMode old = g_mode;
    g_mode = *m;
    *m = old;
    return hipSuccess;
}
}

#define CHECK(c)                                                  \
    do {                                                          \
        if (!(c)) {                                               \
            printf("line %d: %s\n", __LINE__, #c);                \
            exit(1);                                              \
        }                                                         \
    } while (0)

static void write_slot(const SlotUse& u, uint32_t total) {  // what the kernel does
    u.slot->total = total;
    u.slot->total2 = total + 1;
    u.slot->bad_lobes = 3;
    __atomic_store_n(&u.slot->seq, u.seq, __ATOMIC_RELEASE);
}

int main() {
    HostSlots pool;
    uint32_t total = 0, total2 = 0;
    int32_t bad = 0;
    {  // a refused allocation: no slot, and the next call tries again, in the relaxed capture mode
        g_malloc = hipErrorOutOfMemory;
        SlotUse u(pool, nullptr);
        CHECK(!u.slot && g_mallocs == 1);
    }
    g_malloc = hipSuccess;
    for (int i = 0; i < 200; ++i) {  // calls that are waited for
        SlotUse u(pool, nullptr);
        CHECK(u.slot && u.seq != 0);
        write_slot(u, 7 + i);
        CHECK(u.wait(&total, &bad, &total2) == hipSuccess && total == 7u + i && total2 == 8u + i && bad == 3 && !u.slot);
    }
    CHECK(g_mallocs == 2 && g_mode_at_malloc == hipStreamCaptureModeRelaxed && g_mode == hipStreamCaptureModeGlobal);
    CHECK(g_syncs == 0);
    for (int i = 0; i < 200; ++i) {  // calls that end before they wait: the stream is waited for, the slot given back
        SlotUse u(pool, nullptr);
        CHECK(u.slot);
    }
    CHECK(g_syncs == 200);
    for (int i = 0; i < 200; ++i) {  // a word that never comes: an error, and the slot comes back (the stream is idle)
        SlotUse u(pool, nullptr);
        CHECK(u.slot && (i > 1 || u.wait(&total, &bad) == hipErrorUnknown));
    }
    {  // all slots lent: none for the next call
        SlotUse* lent[64];
        for (auto& u : lent) {
            u = new SlotUse(pool, nullptr);
            CHECK(u->slot);
        }
        SlotUse none(pool, nullptr);
        CHECK(!none.slot);
        for (auto& u : lent) delete u;
    }
    {  // no slot while the stream is captured, or where that cannot be asked
        g_status = hipStreamCaptureStatusActive;
        SlotUse a(pool, nullptr);
        CHECK(!a.slot);
        g_status = hipStreamCaptureStatusNone;
        g_capturing = hipErrorStreamCaptureImplicit;
        SlotUse b(pool, nullptr);
        CHECK(!b.slot);
        g_capturing = hipSuccess;
    }
    g_sync = hipErrorLaunchFailure;
    for (int i = 0; i < 64; ++i) {  // the stream cannot be waited for: a kernel might still write, the slot stays out
        SlotUse u(pool, nullptr);
        CHECK(u.slot);
    }
    SlotUse u(pool, nullptr);
    CHECK(!u.slot);
    return 0;
}
