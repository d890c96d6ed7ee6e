// Content-addressed caches of symbol-side plans.
#pragma once

#include <cstdint>
#include <cstring>
#include <initializer_list>
#include <memory>
#include <mutex>
#include <unordered_map>
#include <utility>
#include <vector>

namespace dol {

// Hash of a key, eight bytes at a time (a byte-wise hash of a kilobyte of symbol ids costs as much as a launch): multiply,
// fold the high half down, finish with one more round (multiplier and fold by 32 as in the published 64-bit mixer degski64,
// the start is 2^64 over the golden ratio).  Equal keys are compared byte by byte, so only speed rests on it.
inline uint64_t hash_bytes(const void *data, size_t n)
{
    const unsigned char *p = static_cast<const unsigned char *>(data);
    uint64_t h = 0x9E3779B97F4A7C15ull ^ n;
    auto mix = [&h](uint64_t w) {
        h = (h ^ w) * 0xD6E8FEB86659FD93ull;
        h ^= h >> 32;
    };
    for (; n >= 8; n -= 8, p += 8) {
        uint64_t w;
        std::memcpy(&w, p, 8);
        mix(w);
    }
    uint64_t w = 0;
    std::memcpy(&w, p, n);
    mix(w);
    mix(0);
    return h;
}

// At most kCacheMax plans per cache: a program whose predicates or symbol lists keep changing would otherwise grow the
// caches without bound.  Beyond that the plan that has gone unused longest is released (hipFree waits for launches
// that may still read its arrays; plans handed out earlier must not be used after kCacheMax newer ones were made).
constexpr size_t kCacheMax = 4096;

template <typename Plan>
struct Cache {
    struct Entry {
        std::vector<unsigned char> key;
        std::unique_ptr<Plan> plan;
        uint64_t used = 0;
    };
    std::mutex mu;
    std::unordered_multimap<uint64_t, Entry> map;
    uint64_t clock = 0;

    const Plan *find(uint64_t h, const std::vector<unsigned char> &key)
    {
        auto range = map.equal_range(h);
        for (auto it = range.first; it != range.second; ++it)
            if (it->second.key == key) { it->second.used = ++clock; return it->second.plan.get(); }
        return nullptr;
    }
    const Plan *insert(uint64_t h, std::vector<unsigned char> &&key, std::unique_ptr<Plan> &&plan)
    {
        if (map.size() >= kCacheMax) {
            auto oldest = map.begin();
            for (auto it = map.begin(); it != map.end(); ++it)
                if (it->second.used < oldest->second.used) oldest = it;
            map.erase(oldest);
        }
        auto it = map.emplace(h, Entry{std::move(key), std::move(plan), ++clock});
        return it->second.plan.get();
    }
};

inline std::vector<unsigned char> make_key(int device, std::initializer_list<std::pair<const void *, size_t>> parts)
{
    size_t total = sizeof(int);
    for (const auto &p : parts) total += sizeof(uint64_t) + p.second;
    std::vector<unsigned char> key(total);
    unsigned char *at = key.data();
    std::memcpy(at, &device, sizeof(int));
    at += sizeof(int);
    for (const auto &p : parts) {
        const uint64_t n = p.second;
        std::memcpy(at, &n, sizeof n);
        at += sizeof n;
        if (n) std::memcpy(at, p.first, n);
        at += n;
    }
    return key;
}

}  // namespace dol
