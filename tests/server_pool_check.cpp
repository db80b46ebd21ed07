// Host check of lp_server_pool.h with a memory that records what it is asked for: no GPU code.
#include <cassert>
#include <cstdio>
#include <cstdlib>
#include <string>
#include <vector>

#include "lp_server_pool.h"

namespace {

struct Log {
    std::vector<std::string> calls;
    int next_wait = 0;  // result of the next wait
    size_t limit = ~size_t(0), in_use = 0;
};

struct FakeMemory {
    using Error = int;
    using Stream = int;
    using Pinned = double;
    Log* log;
    static int ok() { return 0; }
    static bool out_of_memory(int e) { return e == 2; }
    int allocate(char** out, size_t bytes) {
        if (log->in_use + bytes > log->limit) return 2;
        log->in_use += bytes;
        *out = static_cast<char*>(std::malloc(bytes));
        log->calls.push_back("allocate " + std::to_string(bytes));
        return 0;
    }
    void release(char* p) {
        std::free(p);
        log->calls.push_back("release");
    }
    int allocate_pinned(double** out) {
        *out = new double;
        return 0;
    }
    void release_pinned(double* p) { delete p; }
    int wait(int s) {
        log->calls.push_back("wait " + std::to_string(s));
        return log->next_wait;
    }
};

#define CHECK(c) \
    do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); std::exit(1); } } while (0)

// A block of a failed set-up is waited for on that set-up's stream before anything can take it.
void failed_setup() {
    Log log;
    {
        lpgpu::ServerPool<FakeMemory> pool(1000, FakeMemory{&log});
        char *a = nullptr, *b = nullptr;
        size_t held = 0;
        CHECK(pool.admit(100) && pool.take(100, &a, &held) == 0 && held == 100);
        CHECK(pool.give_unfinished(7, a, held, 100));
        pool.retire(100);
        CHECK(log.calls.size() == 2 && log.calls[1] == "wait 7");
        CHECK(pool.admit(100) && pool.take(100, &b, &held) == 0 && b == a);  // reused after the wait
        // the wait fails: freed, not kept
        log.next_wait = 1;
        CHECK(!pool.give_unfinished(8, b, held, 100));
        pool.retire(100);
        CHECK(log.calls.size() == 4 && log.calls[2] == "wait 8" && log.calls[3] == "release");
        CHECK(pool.admit(1000) && pool.take(1000, &a, &held) == 0);  // nothing of it counts any more
        CHECK(log.calls.back() == "allocate 1000");
        pool.give(a, held, 1000);
        pool.retire(1000);
        // no allocation was made before the failure: only the wait
        CHECK(!pool.give_unfinished(9, nullptr, 0, 500));
        CHECK(log.calls.back() == "wait 9" && pool.admit(1000));
    }
    CHECK(log.calls.back() == "release");
}

}  // namespace

int main() {
    failed_setup();
    std::puts("ok");
    return 0;
}
