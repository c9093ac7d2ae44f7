// Batches on the two-device runtime of this folder: the library's scheduler with launchers that
// only note where they were sent.  Exits with the line of the first check that fails, modulo 256.
#include <cstdio>
#include <memory>
#include <new>
#include <set>
#include <string>

#include "pond_handle.h"

using namespace pond;

#define CHECK(x)                                               \
    do {                                                       \
        if (!(x)) {                                            \
            std::printf("line %d: %s\n", __LINE__, #x);        \
            std::exit(__LINE__ % 256 ? __LINE__ % 256 : 1);    \
        }                                                      \
    } while (0)

// memory for C++ objects that has run out while a capture is open
static bool memory_short = false;
void *operator new(size_t n)
{
    if (memory_short && fake::captures) throw std::bad_alloc();
    if (void *p = std::malloc(n)) return p;
    throw std::bad_alloc();
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

static int launches, elsewhere;
static hipError_t launched(const LaunchCtx &c)
{
    ++launches;
    if (fake::device_of(c.st) != 0) ++elsewhere; // the members' memory is on device 0
    return hipSuccess;
}
namespace pond {
hipError_t launch_stream(const LaunchCtx &c, const SlotDesc *, int, int) { return launched(c); }
hipError_t launch_force_collide(const LaunchCtx &c, const SlotDesc *, int, int) { return launched(c); }
hipError_t launch_step_fused(const LaunchCtx &c, const SlotDesc *, int, int) { return launched(c); }
hipError_t launch_collide_check(const LaunchCtx &, const SlotDesc *, int, int) { return hipSuccess; }
hipError_t launch_reset_slot_flags(hipStream_t, const SlotDesc *, int) { return hipSuccess; }
hipError_t launch_gather_slot_flags(hipStream_t, const SlotDesc *, int, int *) { return hipSuccess; }
int handle_fail(pond_handle *, int code, const char *, ...) { return code; }
int handle_finish_batch(pond_handle *h, const int *, int nsteps) { return h->steps += nsteps, POND_OK; }
} // namespace pond

// a member of its own group
static std::unique_ptr<pond_handle> member(int tile, bool fused)
{
    std::unique_ptr<pond_handle> h(new pond_handle());
    h->lc = LaunchCtx{2, 64, 64, 4096, 0, nullptr, tile};
    h->lc.fused = fused;
    h->initialised = true;
    h->st_tiles = h->fc_tiles = 16 * (1 + tile);
    return h;
}

// a batch on device 0 of `groups` groups, stepped while `current` is the current device; its long
// runs take `side_by_side` streams
static void step(int groups, bool fused, int current, int side_by_side)
{
    const int streams = fake::streams, events = fake::events;
    pond_batch *b = nullptr;
    fake::device = 0;
    CHECK(pond_batch_create(nullptr, &b) == POND_OK);
    std::unique_ptr<pond_handle> h[6];
    for (int i = 0; i < groups; ++i) {
        h[i] = member(i, fused);
        CHECK(pond_batch_add(b, h[i].get()) == POND_OK);
    }
    fake::device = current;
    const int run = fused ? kFusedRun : 2 * kRunPairs;
    for (int change = 0; change < 3; ++change) {
        launches = elsewhere = 0;
        fake::graph_launches.clear();
        CHECK(pond_batch_step(b, 2 * run) == POND_OK);
        const std::set<hipStream_t> used(fake::graph_launches.begin(), fake::graph_launches.end());
        CHECK((int)used.size() == side_by_side && (int)fake::graph_launches.size() == 2 * side_by_side);
        for (hipStream_t st : used) CHECK(st->device == 0);
        CHECK(launches == run * groups * (fused ? 1 : 2) && elsewhere == 0);
        CHECK(fake::device == current && fake::captures == 0);
        CHECK(pond_batch_remove(b, h[0].get()) == POND_OK && pond_batch_add(b, h[0].get()) == POND_OK);
    }
    for (int i = 0; i < groups; ++i) CHECK(h[i]->steps == 3 * 2 * run);
    CHECK(pond_batch_destroy(b) == POND_OK);
    CHECK(fake::streams == streams && fake::events == events);
    fake::device = 0;
}

// the streams of a batch are of its own device, whichever is current
static void device()
{
    for (int current : {0, 1})
        for (bool fused : {true, false})
            for (int groups : {1, 2, 3, 6}) step(groups, fused, current, groups < 3 ? groups : 3);
}

// with fewer streams or events than asked for, fewer groups run side by side
static void shortage()
{
    for (int left : {0, 1, 2}) {
        fake::streams_left = 2 + left; // (the batch's own two)
        step(4, true, 0, 1 + left);
    }
    fake::streams_left = 1 << 30;
    for (int left : {0, 1, 2, 3}) {
        fake::events_left = left; // one to fork, one to join each stream
        step(4, true, 0, left < 2 ? 1 : left);
    }
}

// a capture allocates nothing of its own: an exception there would leave the C entry with the
// capture open
static void memory()
{
    memory_short = true;
    for (bool fused : {true, false}) step(6, fused, 0, 3);
}

int main(int, char **argv)
{
    const std::string what = argv[1];
    if (what == "device") device();
    else if (what == "shortage") shortage();
    else if (what == "memory") memory();
    else return 255;
    return 0;
}
