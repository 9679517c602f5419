// A device array of work items with their count (an int) behind the last.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace sllg {

template <typename Item>
struct ItemList {
    Item* d = nullptr;
    int64_t cap = 0;   // items d holds; 0 while there is none

    // Room for n items; alloc(bytes) returns device memory or throws,
    // release(p) frees it.  When alloc throws the list is empty, so that no
    // launch finds a capacity without its memory.
    template <typename Alloc, typename Release>
    void reserve(int64_t n, Alloc&& alloc, Release&& release)
    {
        if (n <= cap)
            return;
        const int64_t want = std::max<int64_t>(n, 2 * cap);
        clear(release);
        d = static_cast<Item*>(alloc(sizeof(Item) * (size_t)want + sizeof(int)));
        cap = want;
    }
    template <typename Release>
    void clear(Release&& release)
    {
        if (d)
            release(d);
        d = nullptr;
        cap = 0;
    }
    int* count() const { return reinterpret_cast<int*>(reinterpret_cast<char*>(d) + sizeof(Item) * (size_t)cap); }
};

}  // namespace sllg
