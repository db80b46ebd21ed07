// Memory of a server's requests: device allocations and pinned scalar blocks kept for the next
// ones. hipMalloc and hipFree per request cost more than the set-up of a small LP, and hipFree
// waits for every stream of the device. Host code without HIP types: `Memory` allocates, frees
// and waits (HipMemory in the library, a recording one in its host check).
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <mutex>
#include <utility>
#include <vector>

namespace lpgpu {

// Memory is returned only after its last work was waited for, so any stream may take it next.
// Requests are admitted here: the footprints admitted, what reused blocks exceed theirs by and
// the free blocks stay within the budget. A block is reused for a request that needs at least
// 8/9 of it: a small request in a large block would keep the next large one from being
// admitted. A server without requests trims the free blocks to kept(); everything is given back
// when the server and its requests are gone.
template <class Memory>
class ServerPool {
public:
    using Error = typename Memory::Error;
    using Stream = typename Memory::Stream;
    using Pinned = typename Memory::Pinned;

    explicit ServerPool(int64_t budget, Memory memory = Memory()) : memory_(memory), budget_(budget) {}
    ~ServerPool() {
        for (auto& f : free_) memory_.release(f.first);
        for (Pinned* p : pinned_) memory_.release_pinned(p);
    }
    ServerPool(const ServerPool&) = delete;
    ServerPool& operator=(const ServerPool&) = delete;

    // What a server without requests keeps for the next ones: the footprints of some hundred LPs of
    // a few thousand rows, little beside the device's memory or the budget.
    int64_t kept() const { return std::min<int64_t>(budget_ / 8, int64_t(256) << 20); }

    bool admit(size_t need) {
        std::lock_guard<std::mutex> lk(mu_);
        if (admitted_ + over_ + static_cast<int64_t>(need) > budget_) return false;
        admitted_ += static_cast<int64_t>(need);
        return true;
    }
    void retire(size_t need) {
        std::lock_guard<std::mutex> lk(mu_);
        admitted_ -= static_cast<int64_t>(need);
    }
    // Memory for an admitted request: a free block (*held bytes of it) or a new one. Nothing is
    // allocated or released under the lock: a release waits for the whole device, and admit() is
    // called with the server's own lock held.
    Error take(size_t need, char** out, size_t* held) {
        std::vector<char*> drop;
        {
            std::lock_guard<std::mutex> lk(mu_);
            size_t best = free_.size();
            for (size_t i = 0; i < free_.size(); ++i)
                if (free_[i].second >= need && free_[i].second - need <= need / 8 && (best == free_.size() || free_[i].second < free_[best].second)) best = i;
            if (best < free_.size() && admitted_ + over_ + static_cast<int64_t>(free_[best].second - need) <= budget_) {
                *out = free_[best].first;
                *held = free_[best].second;
                free_bytes_ -= static_cast<int64_t>(*held);
                taken_ += static_cast<int64_t>(*held);
                over_ += static_cast<int64_t>(*held - need);
                free_.erase(free_.begin() + static_cast<std::ptrdiff_t>(best));
                return Memory::ok();
            }
            while (!free_.empty() && taken_ + free_bytes_ + static_cast<int64_t>(need) > budget_) drop.push_back(detach());
            taken_ += static_cast<int64_t>(need);
        }
        for (char* p : drop) memory_.release(p);
        Error e = memory_.allocate(out, need);
        while (Memory::out_of_memory(e)) {
            char* p = nullptr;
            {
                std::lock_guard<std::mutex> lk(mu_);
                if (!free_.empty()) p = detach();
            }
            if (!p) break;
            memory_.release(p);
            e = memory_.allocate(out, need);
        }
        if (e == Memory::ok()) {
            *held = need;
        } else {
            std::lock_guard<std::mutex> lk(mu_);
            taken_ -= static_cast<int64_t>(need);
        }
        return e;
    }
    // Releases free blocks, the largest first, until they hold at most `bytes`.
    void trim(int64_t bytes) {
        std::vector<char*> drop;
        {
            std::lock_guard<std::mutex> lk(mu_);
            if (free_bytes_ <= bytes) return;
            std::sort(free_.begin(), free_.end(), [](const auto& a, const auto& b) { return a.second < b.second; });
            while (free_bytes_ > bytes) drop.push_back(detach());
        }
        for (char* p : drop) memory_.release(p);
    }
    // The last work on p was waited for.
    void give(char* p, size_t held, size_t need) {
        std::lock_guard<std::mutex> lk(mu_);
        forget(held, need);
        free_bytes_ += static_cast<int64_t>(held);
        free_.emplace_back(p, held);
    }
    // p of a set-up that failed part way: copies and kernels on it may still be queued on s. They
    // are waited for; where that fails too the block is freed (which waits for the device), not
    // kept. Returns whether s was waited for.
    bool give_unfinished(Stream s, char* p, size_t held, size_t need) {
        const bool done = memory_.wait(s) == Memory::ok();
        if (!p) return done;
        if (done) {
            give(p, held, need);
            return true;
        }
        memory_.release(p);
        std::lock_guard<std::mutex> lk(mu_);
        forget(held, need);
        return false;
    }
    Error take_pinned(Pinned** out) {
        {
            std::lock_guard<std::mutex> lk(mu_);
            if (!pinned_.empty()) {
                *out = pinned_.back();
                pinned_.pop_back();
                return Memory::ok();
            }
        }
        return memory_.allocate_pinned(out);
    }
    void give_pinned(Pinned* p) {
        std::lock_guard<std::mutex> lk(mu_);
        pinned_.push_back(p);
    }

private:
    void forget(size_t held, size_t need) {
        taken_ -= static_cast<int64_t>(held);
        over_ -= static_cast<int64_t>(held - need);
    }
    // A free block that no longer counts, to be released without the lock.
    char* detach() {
        char* p = free_.back().first;
        free_bytes_ -= static_cast<int64_t>(free_.back().second);
        free_.pop_back();
        return p;
    }
    Memory memory_;
    std::mutex mu_;
    int64_t budget_, admitted_ = 0, over_ = 0, taken_ = 0, free_bytes_ = 0;
    std::vector<std::pair<char*, size_t>> free_;
    std::vector<Pinned*> pinned_;
};

}  // namespace lpgpu
