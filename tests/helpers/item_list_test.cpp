// Host test of the device work lists: an allocation that fails leaves the
// list empty and the next one starts afresh.
#include <cstdio>
#include <cstdlib>
#include <new>

#include "item_list.hpp"

struct Item {
    int a, b, c;
};

static int live = 0;
static bool broken = false;

static void* take(size_t bytes)
{
    if (broken)
        throw std::bad_alloc();
    ++live;
    return std::malloc(bytes);
}
static void give(void* p)
{
    --live;
    std::free(p);
}

#define CHECK(x)                                         \
    if (!(x)) {                                          \
        std::printf("line %d: %s\n", __LINE__, #x);      \
        return 1;                                        \
    }

int main()
{
    sllg::ItemList<Item> l;
    l.reserve(5, take, give);
    CHECK(l.d && l.cap == 5 && live == 1);
    *l.count() = 5;
    CHECK((char*)l.count() == (char*)l.d + 5 * sizeof(Item));
    broken = true;
    bool thrown = false;
    try {
        l.reserve(9, take, give);
    } catch (const std::bad_alloc&) {
        thrown = true;
    }
    CHECK(thrown && !l.d && l.cap == 0 && live == 0);   // nothing to launch with
    thrown = false;
    try {
        l.reserve(1, take, give);                       // still too small for one item
    } catch (const std::bad_alloc&) {
        thrown = true;
    }
    CHECK(thrown && !l.d);
    broken = false;
    l.reserve(9, take, give);
    CHECK(l.d && l.cap == 9 && live == 1);
    l.reserve(10, take, give);
    CHECK(l.cap == 18 && live == 1);
    l.clear(give);
    CHECK(!l.d && l.cap == 0 && live == 0);
    std::puts("ok");
    return 0;
}
