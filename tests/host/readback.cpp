// Read-backs on the two-device runtime of this folder; exits with the line of the first check
// that fails, modulo 256.
#include <cstdio>
#include <string>
#include <vector>

#include "pond_readback.h"

using namespace pond;

#define CHECK(x)                                               \
    do {                                                       \
        if (!(x)) {                                            \
            std::printf("line %d: %s\n", __LINE__, #x);        \
            std::exit(__LINE__ % 256 ? __LINE__ % 256 : 1);    \
        }                                                      \
    } while (0)

static hipStream_t stream_on(int device)
{
    hipStream_t s;
    fake::device = device;
    CHECK(hipStreamCreateWithFlags(&s, hipStreamNonBlocking) == hipSuccess);
    fake::device = 0;
    return s;
}

// five fields of n doubles from the "device" into `dst`, of which those not NULL are read
static void read(size_t n, hipStream_t st, std::vector<double *> dst, hipError_t want = hipSuccess)
{
    std::vector<double> src(5 * n);
    auto form = [&](double *out) {
        for (size_t i = 0; i < src.size(); ++i) out[i] = 0.5 + (double)i;
        return hipSuccess;
    };
    const int before = fake::device;
    fake::copies.clear();
    ReadBack rb;
    for (int i = 0; i < 5; ++i)
        if (dst[i]) rb.add(dst[i], src.data() + i * n, n);
    CHECK(rb.run(st, src.data(), src.size(), form) == want);
    CHECK(fake::device == before); // the caller's current device is its own
    for (int i = 0; i < 5 && want == hipSuccess; ++i)
        for (size_t k = 0; dst[i] && k < n; ++k) CHECK(dst[i][k] == 0.5 + (double)(i * n + k));
}

struct Arrays {
    std::vector<std::vector<double>> a;
    explicit Arrays(size_t n) : a(5, std::vector<double>(n, -1.0)) {}
    std::vector<double *> all()
    {
        std::vector<double *> p;
        for (auto &v : a) p.push_back(v.data());
        return p;
    }
};

constexpr size_t kSmall = 1000, kMiddle = 200000, kLarge = 700001; // one piece, runtime copies, pieces

// a stream of a device that is not the caller's current one
static void device()
{
    for (size_t n : {kSmall, kMiddle, kLarge})
        for (int current : {0, 1}) {
            hipStream_t st = stream_on(1 - current);
            fake::device = current;
            read(n, st, Arrays(n).all());
            read(n, hipStreamPerThread, Arrays(n).all());
            hipStreamDestroy(st);
        }
    CHECK(fake::events == 0);
}

// a helper that cannot have what it needs leaves its pieces to the others
static void events()
{
    hipStream_t st = stream_on(0);
    for (int left : {3, 1, 0}) {
        fake::events_left = left;
        read(kLarge, st, Arrays(kLarge).all());
        CHECK(fake::events == 0);
    }
    hipStreamDestroy(st);
}

// device arrays, which the runtime's copies take too, are not written by the host
static void on_device()
{
    hipStream_t st = stream_on(0);
    double *dev = nullptr;
    CHECK(hipMalloc((void **)&dev, kLarge * sizeof(double)) == hipSuccess);
    for (size_t n : {kSmall, kMiddle, kLarge}) {
        Arrays host(n);
        std::vector<double *> dst = host.all();
        dst[2] = dev;
        read(n, st, dst);
        bool copied = false;
        for (const auto &c : fake::copies) copied = copied || (c.dst == (const char *)dev && c.bytes == n * sizeof(double));
        CHECK(copied);
    }
    hipFree(dev);
    hipStreamDestroy(st);
}

// page-locked arrays are copied into directly, the others beside them through the staging
static void locked()
{
    hipStream_t st = stream_on(0);
    double *pin = nullptr;
    CHECK(hipHostMalloc((void **)&pin, 3 * kLarge * sizeof(double), hipHostMallocDefault) == hipSuccess);
    Arrays other(kLarge);
    auto copied_whole = [](const double *dst) {
        for (const auto &c : fake::copies)
            if (c.dst == (const char *)dst) return c.bytes == kLarge * sizeof(double);
        return false;
    };
    std::vector<double *> dst = other.all();
    dst[1] = pin, dst[3] = pin + kLarge;
    read(kLarge, st, dst); // three fields of pageable memory are above the staging still
    CHECK(copied_whole(dst[1]) && copied_whole(dst[3]) && !copied_whole(dst[0]));
    dst[0] = pin + 2 * kLarge;
    read(kLarge, st, dst); // two are within it: the runtime's copies
    for (double *d : dst) CHECK(copied_whole(d));
    read(kLarge, st, {pin, pin + kLarge, pin + 2 * kLarge, nullptr, nullptr});
    CHECK(fake::copies.size() == 3);
    hipHostFree(pin);
    hipStreamDestroy(st);
}

// all fields of a small lattice are formed in the staging: no copy
static void small()
{
    hipStream_t st = stream_on(0);
    Arrays a(kSmall), b(100000);
    read(kSmall, st, a.all());
    CHECK(fake::copies.empty());
    read(kSmall, st, {a.all()[0], nullptr, nullptr, a.all()[3], nullptr});
    CHECK(fake::copies.empty());
    read(100000, st, {nullptr, b.all()[1], b.all()[2], nullptr, nullptr}); // two of a larger one: one copy
    CHECK(fake::copies.size() == 1 && fake::within(fake::pinned, fake::copies[0].dst));
    hipStreamDestroy(st);
}

// a process of one core has no helper: the runtime's copies, not one piece after another
static void one_core()
{
    hipStream_t st = stream_on(0);
    read(kLarge, st, Arrays(kLarge).all());
    CHECK(fake::copies.size() == 5);
    hipStreamDestroy(st);
}

int main(int, char **argv)
{
    const std::string what = argv[1];
    g_stage.enter();
    if (what == "device") device();
    else if (what == "events") events();
    else if (what == "locked") locked();
    else if (what == "on_device") on_device();
    else if (what == "small") small();
    else if (what == "one_core") return one_core(), 0;
    else return 255;
    CHECK(!fake::pinned.empty());
    g_stage.leave();
    CHECK(fake::pinned.empty() && fake::streams == 0);
    return 0;
}
