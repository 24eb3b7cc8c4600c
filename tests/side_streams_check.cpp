// Checks of rt_side_streams.h without a GPU: streams are numbers, a stream is idle unless it is in `busy`.
#include "rt_side_streams.h"

#include <cstdio>
#include <cstring>
#include <set>

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
void Fake::destroy(int, int st) { destroyed.insert(st); }

int next_stream = 100, failures = 0;
void check(bool ok, const char *what)
{
    if (!ok) { std::printf("FAILED %s\n", what); ++failures; }
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
    for (int i = 0; i < 3; ++i) pool.count_context(-1);
}
}  // namespace

int main(int argc, char **argv)
{
    if (argc != 2) return 2;
    if (!std::strcmp(argv[1], "unrelated_callers")) unrelated_callers();
    else return 2;
    return failures ? 1 : 0;
}
