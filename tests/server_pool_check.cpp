// Host check of lp_server_pool.h with a memory that records what it is asked for: no GPU code.
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <future>
#include <string>
#include <vector>

#include "lp_server_pool.h"

namespace {

struct Log {
    std::vector<std::string> calls;
    int next_wait = 0;  // result of the next wait
    size_t limit = ~size_t(0), in_use = 0;
    std::function<void()> during;  // run inside every allocation and release
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
        if (log->during) log->during();
        log->in_use += bytes;
        *out = static_cast<char*>(std::malloc(bytes));
        log->calls.push_back("allocate " + std::to_string(bytes));
        return 0;
    }
    void release(char* p) {
        if (log->during) log->during();
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

// While a block is allocated, and while others are released for it, the pool answers other threads.
void no_memory_call_under_the_lock() {
    Log log;
    lpgpu::ServerPool<FakeMemory> pool(1000, FakeMemory{&log});
    int calls = 0;
    log.during = [&] {
        ++calls;
        auto other = std::async(std::launch::async, [&] {
            const bool in = pool.admit(1);
            if (in) pool.retire(1);
        });
        if (other.wait_for(std::chrono::seconds(5)) != std::future_status::ready) {
            std::puts("the pool is locked during a memory call");
            std::_Exit(1);
        }
    };
    char* p[3];
    size_t held = 0;
    for (char*& q : p) CHECK(pool.admit(300) && pool.take(300, &q, &held) == 0);
    for (char* q : p) pool.give(q, 300, 300), pool.retire(300);
    CHECK(calls == 3);
    // 900 free bytes of 1000: two blocks go before 600 new ones come
    char* big = nullptr;
    CHECK(pool.admit(600) && pool.take(600, &big, &held) == 0 && held == 600);
    CHECK(calls == 6);
    log.during = nullptr;
    pool.give(big, held, 600);
    pool.retire(600);
}

// An allocation that fails counts nothing; free blocks go first when the device is out of memory.
void out_of_memory() {
    Log log;
    lpgpu::ServerPool<FakeMemory> pool(1000, FakeMemory{&log});
    char *a = nullptr, *b = nullptr;
    size_t held = 0;
    CHECK(pool.admit(300) && pool.take(300, &a, &held) == 0);
    pool.give(a, held, 300);
    pool.retire(300);
    log.limit = 0;
    CHECK(pool.admit(400) && pool.take(400, &b, &held) == 2);
    CHECK(log.calls.back() == "release");
    pool.retire(400);
    log.limit = ~size_t(0);
    CHECK(pool.admit(1000) && pool.take(1000, &b, &held) == 0);
    pool.give(b, held, 1000);
    pool.retire(1000);
}

// A server without requests keeps at most kept(): an eighth of its budget, 256 MB at most.
void idle() {
    Log log;
    lpgpu::ServerPool<FakeMemory> pool(1000, FakeMemory{&log});
    CHECK(pool.kept() == 125);
    CHECK(lpgpu::ServerPool<FakeMemory>(int64_t(1) << 40, FakeMemory{&log}).kept() == 256 << 20);
    char* p[4];
    const size_t sizes[4] = {90, 400, 30, 200};
    size_t held = 0;
    for (int i = 0; i < 4; ++i) CHECK(pool.admit(sizes[i]) && pool.take(sizes[i], &p[i], &held) == 0);
    for (int i = 0; i < 4; ++i) pool.give(p[i], sizes[i], sizes[i]), pool.retire(sizes[i]);
    log.calls.clear();
    pool.trim(pool.kept());
    CHECK(log.calls.size() == 2);  // 400 and 200; 90 + 30 stay
    pool.trim(pool.kept());
    CHECK(log.calls.size() == 2);
    char* q = nullptr;
    CHECK(pool.admit(30) && pool.take(30, &q, &held) == 0 && q == p[2]);
    CHECK(pool.admit(85) && pool.take(85, &q, &held) == 0 && q == p[0] && held == 90);
}

// A small request does not take a large block, which would keep a large request out.
void no_small_request_in_a_large_block() {
    Log log;
    lpgpu::ServerPool<FakeMemory> pool(1000, FakeMemory{&log});
    char *a = nullptr, *b = nullptr;
    size_t held = 0;
    CHECK(pool.admit(600) && pool.take(600, &a, &held) == 0);
    pool.give(a, held, 600);
    pool.retire(600);
    CHECK(pool.admit(100) && pool.take(100, &b, &held) == 0 && held == 100);
    CHECK(pool.admit(900));
    CHECK(pool.take(900, &a, &held) == 0 && held == 900);
}

}  // namespace

int main() {
    failed_setup();
    no_memory_call_under_the_lock();
    out_of_memory();
    idle();
    no_small_request_in_a_large_block();
    std::puts("ok");
    return 0;
}
