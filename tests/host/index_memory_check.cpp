// Book-keeping of the index memory against a made-up runtime; run with the name of a check.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <thread>
#include <vector>

#include "index_memory.cpp"

using namespace lsh;

static bool refuse = false;  // operator new fails
void *operator new(std::size_t n) {
    if (refuse) throw std::bad_alloc();
    if (void *p = std::malloc(n)) return p;
    throw std::bad_alloc();
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }

static int failed = 0;
#define CHECK(x) \
    do { \
        if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); ++failed; } \
    } while (0)

static const hipStream_t s = reinterpret_cast<hipStream_t>(uintptr_t(64));
constexpr size_t MB = size_t(1) << 20;

static IndexBlock take(size_t bytes, bool scratch) {
    IndexBlock b;
    CHECK(index_memory_take(0, bytes, scratch, s, b));
    CHECK(b.ptr && b.bytes >= bytes);
    return b;
}

// what is given back is used again, and all of it is released with the last index
static void reuse() {
    index_memory_enter(0);
    IndexBlock a = take(100 * MB, false), x = take(110 * MB, true);
    index_memory_give_scratch(0, x, s);
    index_memory_enter(0);
    IndexBlock y = take(110 * MB, true);
    CHECK(y.ptr == x.ptr);
    index_memory_give_scratch(0, y, s);
    index_memory_give(0, a);
    index_memory_leave(0);
    CHECK(stub.mallocs == 2 && stub.frees == 0);
    IndexBlock b = take(100 * MB, false);
    CHECK(b.ptr == a.ptr);
    index_memory_give(0, b);
    index_memory_leave(0);
    CHECK(stub.bytes == 0 && stub.events == 0);
}

// nothing throws, whatever the host's allocator does: the callers are C entries
static void no_exceptions() {
    static IndexBlock blocks[600];
    for (int device : {0, 1, 7, 63, 200}) {
        refuse = true;
        index_memory_enter(device);
        refuse = false;  // the made-up runtime needs memory
        for (IndexBlock &b : blocks) CHECK(index_memory_take(device, MB, false, s, b));
        for (IndexBlock &b : blocks) {
            refuse = true;
            index_memory_give(device, b);
            refuse = false;
        }
        IndexBlock x;
        CHECK(index_memory_take(device, 3 * MB, true, s, x));
        refuse = true;
        index_memory_leave(device);
        refuse = false;
        index_memory_give_scratch(device, x, s);
        index_memory_enter(device);
        index_memory_leave(device);
        CHECK(stub.bytes == 0 && stub.events == 0);
    }
}

// a table holds little more than it needs for as long as its index lives; scratch is there for a build only
static void slack() {
    index_memory_enter(0);
    index_memory_give(0, take(100 * MB, false));
    IndexBlock b = take(60 * MB, false);
    CHECK(b.bytes == 60 * MB);
    IndexBlock c = take(90 * MB, false);
    CHECK(c.bytes == 100 * MB && stub.mallocs == 2);
    index_memory_give(0, c);
    IndexBlock x = take(60 * MB, true);
    CHECK(x.ptr == c.ptr);
    index_memory_give_scratch(0, x, s);
    index_memory_give(0, b);
    index_memory_leave(0);
    CHECK(stub.bytes == 0 && stub.events == 0);
}

// beyond the limit the oldest blocks go; a block that alone exceeds it goes by itself
static void limit() {
    index_memory_enter(0);
    IndexBlock b[4];
    for (int i = 0; i < 4; ++i) b[i] = take((300 + 50 * i) * MB, false);  // 1500 MB together
    for (const IndexBlock &i : b) index_memory_give(0, i);
    IndexBlock large = take(3000 * MB, false);
    index_memory_give(0, large);
    CHECK(stub.frees == 1 && stub.bytes == 1500 * MB);
    IndexBlock more = take(700 * MB, false);
    index_memory_give(0, more);  // 2200 MB: the oldest, 300 MB, goes
    CHECK(stub.frees == 2 && stub.bytes == 1900 * MB);
    index_memory_give(0, take(350 * MB, false));
    CHECK(stub.frees == 2);
    index_memory_leave(0);
    CHECK(stub.bytes == 0);
}

int main(int, char **argv) {
    if (!std::strcmp(argv[1], "reuse")) reuse();
    else if (!std::strcmp(argv[1], "no_exceptions")) no_exceptions();
    else if (!std::strcmp(argv[1], "slack")) slack();
    else if (!std::strcmp(argv[1], "limit")) limit();
    else return 2;
    CHECK(stub.wrong == 0);
    return failed != 0;
}
