// table_pool.h on made-up queues: a block is not handed out while work that reads it can still run.
#include "table_pool.h"

#include <stdio.h>

#include <thread>

using namespace bpt;

static int failed = 0;
#define CHECK(...) ((__VA_ARGS__) ? (void)0 : (void)(printf("line %d: %s\n", __LINE__, #__VA_ARGS__), ++failed))

static const std::vector<int32_t> kSmall(10, 1), kLarge(5000, 2);

static TableBlock* take(TablePool& pool, const std::vector<int32_t>& h) {
    TableBlock* b = nullptr;
    CHECK(pool.acquire(h, &b) == hipSuccess && b && b->p && !memcmp(b->p, h.data(), h.size() * 4));
    return b;
}
static void call(TablePool& pool, TableBlock* b, hipStream_t s) {   // a kernel that reads the block, then its event
    ++queue_of(s).put;
    pool.note(*b, s);
}
static void run(hipStream_t s) { queue_of(s).done = queue_of(s).put; }

static void reuse() {
    TablePool pool;
    TableBlock* a = take(pool, kSmall);
    int32_t* const p = a->p;
    call(pool, a, stream(1));
    call(pool, a, stream(2));
    pool.release(a);
    run(stream(1));
    TableBlock* b = take(pool, kSmall);
    CHECK(b->p != p);   // stream 2 still reads it
    pool.release(b);
    run(stream(2));
    TableBlock* c = take(pool, kSmall);
    CHECK(c->p == p && g_waits == 0);
    call(pool, c, stream(1));
    TableBlock* d = take(pool, kLarge);
    CHECK(d->p != p && d->capacity >= kLarge.size());
    pool.release(c);
    pool.release(d);
}

// one handle, two queues: each host thread's own default stream, or a stream made after another was destroyed
static void handles() {
    TablePool pool;
    TableBlock* a = take(pool, kSmall);
    int32_t* const p = a->p;
    call(pool, a, stream(3));
    const std::shared_ptr<Queue> first = g_queue[stream(3)];
    g_queue[stream(3)] = std::make_shared<Queue>();
    call(pool, a, stream(3));
    run(stream(3));
    pool.release(a);
    TableBlock* b = take(pool, kSmall);
    CHECK(b->p != p);   // the first queue still reads it
    pool.release(b);
    first->done = first->put;
    TableBlock* c = take(pool, kSmall);
    CHECK(c->p == p);
    pool.release(c);
}

static void captures() {
    TablePool pool;
    TableBlock* a = take(pool, kSmall);
    int32_t* const p = a->p;
    queue_of(stream(4)).capturing = true;
    call(pool, a, stream(4));
    queue_of(stream(4)).capturing = false;
    run(stream(4));
    call(pool, a, stream(4));
    run(stream(4));
    CHECK(g_memory.count(p));
    pool.release(a);
    CHECK(!g_memory.count(p) && pool.blocks == 0);   // freed with its graph: nobody else gets it

    TableBlock* b = take(pool, kSmall);   // no event: as if captured
    int32_t* const q = b->p;
    g_no_events = true;
    call(pool, b, stream(1));
    g_no_events = false;
    pool.release(b);
    CHECK(!g_memory.count(q));
}

static void many_calls() {
    TablePool pool;
    TableBlock* a = take(pool, kSmall);
    for (size_t i = 0; i < kTableUses; ++i) call(pool, a, stream(5));
    CHECK(!a->unknown && a->events.size() == kTableUses);
    call(pool, a, stream(5));
    CHECK(a->unknown && a->events.size() == kTableUses);
    run(stream(5));
    pool.release(a);
    CHECK(pool.blocks == 0);
}

// more graphs queued than there are blocks: the next one waits for the oldest that is large enough; another thread's
// call does not wait with it
static TablePool* g_pool = nullptr;
static bool g_locked = false;
static void other_thread() {
    std::thread([] {
        if (g_pool->m.try_lock())
            g_pool->m.unlock();
        else
            g_locked = true;
    }).join();
}
static void all_in_use(bool large) {
    TablePool pool;
    g_pool = &pool;
    g_on_wait = other_thread;
    int32_t* first = nullptr;
    for (int i = 0; i < kTableBlocks; ++i) {
        TableBlock* b = take(pool, kSmall);
        if (i == 0) first = b->p;
        call(pool, b, stream(100 + i));
        pool.release(b);
    }
    CHECK(pool.blocks == kTableBlocks && g_waits == 0);
    TableBlock* b = take(pool, large ? kLarge : kSmall);
    CHECK(g_waits >= 1 && pool.blocks == kTableBlocks);
    if (!large) {
        CHECK(b->p == first && queue_of(stream(100)).done == queue_of(stream(100)).put);
        CHECK(queue_of(stream(101)).done < queue_of(stream(101)).put);
    }
    call(pool, b, stream(100));
    // a ninth and a tenth while graphs hold all the others: freed with their graphs
    std::vector<TableBlock*> held = {b};
    for (int i = 1; i < kTableBlocks + 2; ++i) {
        held.push_back(take(pool, kLarge));
        call(pool, held.back(), stream(200 + i));
    }
    CHECK(pool.blocks > kTableBlocks);
    for (TableBlock* x : held) pool.release(x);
    CHECK(pool.blocks == kTableBlocks && (int)pool.free.size() == kTableBlocks);
    CHECK(!g_locked);
    g_on_wait = nullptr;
}

int main(int argc, char** argv) {
    const int which = atoi(argv[1]);
    if (which == 0) reuse();
    if (which == 1) handles();
    if (which == 2) captures();
    if (which == 3) many_calls();
    if (which == 4) all_in_use(false);
    if (which == 5) all_in_use(true);
    CHECK(g_memory.empty());   // a pool leaves nothing behind
    return failed ? 1 : 0;
}
