// host_copy.h against a stub of the runtime: every way through it returns the bytes or an error, and returns.
#include "host_copy.h"

#include <dlfcn.h>
#include <pthread.h>

#include <cstdio>
#include <random>

using namespace legend;

// threads beyond this many cannot be created
static int threads_left = 1 << 30;
extern "C" int pthread_create(pthread_t* t, const pthread_attr_t* a, void* (*f)(void*), void* x) {
    using Fn = int (*)(pthread_t*, const pthread_attr_t*, void* (*)(void*), void*);
    static Fn real = reinterpret_cast<Fn>(dlsym(RTLD_NEXT, "pthread_create"));
    if (threads_left <= 0) return 11;
    --threads_left;
    return real(t, a, f, x);
}

static int failures = 0;
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); ++failures; } } while (0)

struct Job {
    std::vector<std::vector<char>> src;
    std::vector<char> out;
    std::vector<HostCopyPart> parts;
    // sizes in bytes, negative: host memory
    explicit Job(const std::vector<int64_t>& sizes) {
        std::mt19937_64 rng(7);
        size_t total = 0;
        for (int64_t s : sizes) {
            const size_t n = (size_t)(s < 0 ? -s : s);
            src.emplace_back(n);
            for (size_t i = 0; i + 8 <= n; i += 8) { const uint64_t v = rng(); std::memcpy(src.back().data() + i, &v, 8); }
            total += n;
        }
        out.assign(total, 0);
        size_t at = 0;
        for (size_t k = 0; k < sizes.size(); ++k) {
            parts.push_back({out.data() + at, src[k].data(), src[k].size(), sizes[k] >= 0});
            at += src[k].size();
        }
    }
    bool whole() const {
        size_t at = 0;
        for (const auto& s : src) {
            if (std::memcmp(out.data() + at, s.data(), s.size()) != 0) return false;
            at += s.size();
        }
        return true;
    }
};

static void reset() {
    stub.fail_host_malloc = stub.attributes_fail = stub.fail_set_device = 0;
    stub.fail_event_create = stub.fail_copy = stub.fail_sync = -1;
    stub.dst_type = hipMemoryTypeUnregistered;
    stub.copies = stub.syncs = stub.plain = 0;
    threads_left = 1 << 30;
}

int main() {
    const int64_t MB = 1 << 20, lim = (int64_t)HostCopyRing::kMinBytes;
    StubStream stream;
    const std::vector<std::vector<int64_t>> shapes = {
        {lim}, {lim + 4}, {lim + MB - 4}, {MB + 8, -(3 * MB + 12), 30 * MB}, {-lim}, {-(lim + 20), 8}, {20 * MB, -(20 * MB), 20 * MB, -(4 * MB)}};
    {   // the ring: any number of threads, none at all
        for (const auto& s : shapes)
            for (int threads : {1 << 30, 3, 1, 0}) {
                reset();
                HostCopyRing ring;
                Job j(s);
                threads_left = threads;
                CHECK(copy_parts(ring, j.parts, 0, &stream) == hipSuccess);
                CHECK(j.whole());
                CHECK(stub.plain == 0);
                CHECK(copy_parts(ring, j.parts, 0, &stream) == hipSuccess);      // and a second time on the same ring
                ring.release();
                CHECK(stub.host_blocks == 0 && stub.events == 0);
            }
    }
    // plain copies: a destination that is not pageable, a small read, no pinned memory, no events
    for (int why = 0; why < 5; ++why) {
        reset();
        HostCopyRing ring;
        Job j(why == 2 ? std::vector<int64_t>{lim - 4} : std::vector<int64_t>{20 * MB, -(20 * MB), 20 * MB});
        if (why == 0) stub.dst_type = hipMemoryTypeHost;
        if (why == 1) stub.dst_type = hipMemoryTypeDevice;
        if (why == 3) stub.fail_host_malloc = 1;
        if (why == 4) stub.fail_event_create = 3;
        CHECK(copy_parts(ring, j.parts, 0, &stream) == hipSuccess);
        CHECK(j.whole());
        CHECK(stub.plain == (why == 2 ? 1 : 2) && stub.copies == 0);
        CHECK(stub.host_blocks == 0 && stub.events == 0);
        ring.release();
    }
    {   // the runtime does not know the pointer: pageable
        reset();
        HostCopyRing ring;
        Job j({lim});
        stub.attributes_fail = 1;
        CHECK(copy_parts(ring, j.parts, 0, &stream) == hipSuccess && j.whole() && stub.plain == 0);
        ring.release();
    }
    // an error at any point ends the call with that error, with nothing of it left on the stream
    for (int at : {0, 1, 7, 8, 9, 20, 31})
        for (int threads : {1 << 30, 2, 0})
            for (int kind = 0; kind < 3; ++kind) {
                reset();
                HostCopyRing ring;
                Job j({16 * MB, -(4 * MB), 16 * MB});
                (kind == 0 ? stub.fail_copy : stub.fail_sync) = kind == 2 ? -1 : at;
                threads_left = threads;
                if (kind == 2) stub.fail_set_device = 1;
                CHECK(copy_parts(ring, j.parts, 0, &stream) == hipErrorUnknown);
                CHECK(stream.idle());
                reset();
                Job k({lim});
                CHECK(copy_parts(ring, k.parts, 0, &stream) == hipSuccess && k.whole());     // the ring is good for the next call
                ring.release();
            }
    std::printf(failures ? "%d failures\n" : "ok\n", failures);
    return failures != 0;
}
