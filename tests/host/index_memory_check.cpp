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

// scratch beyond the limit is stream-ordered and never kept; what is in use counts
static void scratch_limit() {
    index_memory_enter(0);
    IndexBlock a = take(900 * MB, true), b = take(900 * MB, true), c = take(900 * MB, true);
    CHECK(!a.stream_ordered && !b.stream_ordered && c.stream_ordered);
    index_memory_give_scratch(0, c, s);
    CHECK(stub.frees == 1);
    index_memory_give_scratch(0, a, s);
    IndexBlock t = take(400 * MB, false);
    index_memory_give(0, t);  // 900 kept, 900 in use and 400 more: the 900 kept go
    CHECK(stub.frees == 2 && stub.bytes == 1300 * MB);
    index_memory_give_scratch(0, b, s);
    IndexBlock d = take(900 * MB, true);
    CHECK(d.ptr == b.ptr && !d.stream_ordered);
    index_memory_give_scratch(0, d, s);
    index_memory_leave(0);
    CHECK(stub.bytes == 0 && stub.events == 0);
    index_memory_enter(0);  // nothing is counted any more
    a = take(1000 * MB, true), b = take(1000 * MB, true);
    CHECK(!a.stream_ordered && !b.stream_ordered);
    index_memory_give_scratch(0, a, s);
    index_memory_give_scratch(0, b, s);
    index_memory_leave(0);
    CHECK(stub.bytes == 0 && stub.events == 0);
}

// when memory runs out the kept blocks go before a build is refused, and a refused one leaves no trace
static void out_of_memory() {
    stub.most = 2000 * MB;
    index_memory_enter(0);
    IndexBlock a = take(800 * MB, false), b = take(700 * MB, true);
    index_memory_give(0, a);
    index_memory_give_scratch(0, b, s);
    IndexBlock t = take(1500 * MB, false);  // both go
    CHECK(stub.frees == 2 && stub.events == 0);
    IndexBlock x;
    CHECK(!index_memory_take(0, 1000 * MB, true, s, x) && !x.ptr);
    CHECK(!index_memory_take(0, 1000 * MB, false, s, x) && !x.ptr);
    index_memory_give(0, t);
    index_memory_leave(0);
    CHECK(stub.bytes == 0);
    stub.most = SIZE_MAX;
    index_memory_enter(0);
    a = take(1000 * MB, true), b = take(1000 * MB, true);  // nothing is counted any more
    CHECK(!a.stream_ordered && !b.stream_ordered);
    index_memory_give_scratch(0, a, s);
    index_memory_give_scratch(0, b, s);
    index_memory_leave(0);
    CHECK(stub.bytes == 0 && stub.events == 0);
}

// indexes built and destroyed by several threads: no block is with two of them, and all go in the end
static void threads() {
    static std::mutex in_use_mu;
    static std::map<void *, int> in_use;
    auto hold = [](const IndexBlock &b, int by) {
        std::lock_guard<std::mutex> lock(in_use_mu);
        int &user = in_use[b.ptr];
        if (by && user) ++failed;
        user = by;
    };
    auto work = [&](int seed) {
        for (int i = 0; i < 300; ++i) {
            index_memory_enter(0);
            IndexBlock t, x;
            const size_t n = (size_t)(20 + (seed * 37 + i * 13) % 400) * MB;
            if (!index_memory_take(0, n, false, s, t) || !index_memory_take(0, n + 5 * MB, true, s, x)) ++failed;
            hold(t, seed), hold(x, seed);
            hold(x, 0);
            index_memory_give_scratch(0, x, s);
            hold(t, 0);
            index_memory_give(0, t);
            index_memory_leave(0);
        }
    };
    std::vector<std::thread> all;
    for (int i = 1; i <= 6; ++i) all.emplace_back(work, i);
    for (std::thread &t : all) t.join();
    CHECK(stub.bytes == 0 && stub.events == 0);
}

int main(int, char **argv) {
    if (!std::strcmp(argv[1], "reuse")) reuse();
    else if (!std::strcmp(argv[1], "no_exceptions")) no_exceptions();
    else if (!std::strcmp(argv[1], "slack")) slack();
    else if (!std::strcmp(argv[1], "limit")) limit();
    else if (!std::strcmp(argv[1], "scratch_limit")) scratch_limit();
    else if (!std::strcmp(argv[1], "out_of_memory")) out_of_memory();
    else if (!std::strcmp(argv[1], "threads")) threads();
    else return 2;
    CHECK(stub.wrong == 0);
    return failed != 0;
}
