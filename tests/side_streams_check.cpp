// Checks of rt_side_streams.h without a GPU: streams are numbers, a stream is idle unless it is in `busy`.
#include "rt_side_streams.h"

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <set>
#include <thread>
#include <vector>

namespace {
std::set<int> busy, destroyed;
std::mutex busy_mu;
struct Fake {
    using Stream = int;
    static int per_thread() { return 2; }
    static bool idle(int st)
    {
        std::lock_guard<std::mutex> lock(busy_mu);
        return busy.count(st) == 0;
    }
    static void destroy(int, int st);
};
using Pool = rt::SidePool<Fake, 3>;
Pool pool;
bool in_call = false;

int next_stream = 100, failures = 0;
void check(bool ok, const char *what)
{
    if (!ok) { std::printf("FAILED %s\n", what); ++failures; }
}
void Fake::destroy(int, int st)
{
    check(!in_call, "no stream is destroyed inside a call");
    check(busy.count(st) == 0, "no stream with work queued is destroyed");
    pool.give(pool.take(7, 7));   // hangs if the pool is locked
    destroyed.insert(st);
}
// what a call does: streams where the set has none, work queued on them
Pool::Set *call(int device, int caller)
{
    Pool::Set *s = pool.take(device, caller);
    for (int &st : s->st) {
        if (!st) st = next_stream++;
        std::lock_guard<std::mutex> lock(busy_mu);
        busy.insert(st);
    }
    return s;
}
void ran_dry(const Pool::Set *s)
{
    for (int st : s->st) busy.erase(st);
}

void unrelated_callers()
{
    for (int i = 0; i < 3; ++i) pool.count_context(1);
    Pool::Set *a = call(0, 10);
    pool.give(a);
    check(call(0, 10) == a, "calls that follow one another on a stream take the same set");
    pool.give(a);
    Pool::Set *b = call(0, 11);
    check(b != a, "a set with another stream's work queued is not lent");
    pool.give(b);
    Pool::Set *again = call(0, 10);
    check(again == a, "a stream finds its set behind others");
    pool.give(again);
    Pool::Set *other = call(1, 10);
    check(other != a && other != b, "another device, another set");
    pool.give(other);
    busy.insert(a->st[2]);
    busy.erase(a->st[0]);
    busy.erase(a->st[1]);
    Pool::Set *c = call(0, 12);
    check(c != a && c != b, "one busy stream keeps the set back");
    pool.give(c);
    ran_dry(a);
    Pool::Set *d = call(0, 13);
    check(d == a, "a set that has run dry is lent to any stream");
    pool.give(d);
    Pool::Set *p = call(0, 2);
    const int first = p->st[0];
    pool.give(p);
    Pool::Set *q = call(0, 2);
    check(q->st[0] != first, "hipStreamPerThread is another stream in another thread");
    pool.give(q);
    busy.clear();
    for (int i = 0; i < 3; ++i) pool.count_context(-1);
}
// more calls at once than sets used to be kept
void many_at_once()
{
    constexpr int n = 9;
    for (int i = 0; i < n; ++i) pool.count_context(1);
    in_call = true;
    std::set<int> first;
    for (int round = 0; round < 3; ++round) {
        Pool::Set *s[n];
        for (int i = 0; i < n; ++i) s[i] = call(0, 20 + i);
        std::set<int> now;
        for (int i = 0; i < n; ++i) now.insert(s[i]->st, s[i]->st + 3);
        check(now.size() == 3 * n, "calls at once have streams of their own");
        if (round == 0) first = now;
        check(now == first, "no stream is created anew by later calls");
        for (int i = 0; i < n; ++i) pool.give(s[i]);
    }
    in_call = false;
    check(destroyed.empty(), "nothing is destroyed while its contexts live");
    const std::set<int> all = first;
    busy = {*all.begin()};   // one set is still at work
    for (int i = 0; i < n - 2; ++i) pool.count_context(-1);
    check(destroyed.size() == 3 * (n - 2), "idle sets beyond the number of contexts go with their contexts");
    check(destroyed.count(*all.begin()) == 0, "the busy one stays");
    busy.clear();
    pool.count_context(-1);
    pool.count_context(-1);
    check(std::includes(destroyed.begin(), destroyed.end(), all.begin(), all.end()), "the last context gives everything back");
}

// a set is lent to one call at a time
void threads()
{
    pool.count_context(1);
    std::set<Pool::Set *> lent;
    std::mutex mu;
    std::vector<std::thread> ts;
    for (int i = 0; i < 8; ++i)
        ts.emplace_back([&, i] {
            for (int k = 0; k < 2000; ++k) {
                Pool::Set *s = pool.take(0, i % 3 + 30);
                {
                    std::lock_guard<std::mutex> lock(mu);
                    check(lent.insert(s).second, "a set is lent to one call at a time");
                }
                {
                    std::lock_guard<std::mutex> lock(mu);
                    lent.erase(s);
                }
                pool.give(s);
            }
        });
    for (std::thread &t : ts) t.join();
    pool.count_context(-1);
}
}  // namespace

int main(int argc, char **argv)
{
    if (argc != 2) return 2;
    if (!std::strcmp(argv[1], "unrelated_callers")) unrelated_callers();
    else if (!std::strcmp(argv[1], "many_at_once")) many_at_once();
    else if (!std::strcmp(argv[1], "threads")) threads();
    else return 2;
    return failures ? 1 : 0;
}
