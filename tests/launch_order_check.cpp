// Checks of rt_launch_order.h without a GPU: streams are numbers, what is done to them is written down.
#include "rt_launch_order.h"

#include <atomic>
#include <cstdio>
#include <cstring>
#include <set>
#include <string>
#include <thread>
#include <vector>

namespace {
std::string done;
std::set<int> in_capture;
int events = 0;
struct Fake {
    using Stream = int;
    using Event = int;
    static int per_thread() { return 2; }
    static bool capturing(int st) { return in_capture.count(st) != 0; }
    static bool create(int *e) { *e = 1; ++events; return true; }
    static bool record(int, int st) { done += "r" + std::to_string(st) + " "; return st != 66; }
    static bool wait(int st, int) { done += "w" + std::to_string(st) + " "; return true; }
    static void destroy(int) { --events; }
};
using Order = rt::LaunchOrder<Fake, 4>;
int failures = 0;
void check(bool ok, const char *what)
{
    if (!ok) { std::printf("FAILED %s (%s)\n", what, done.c_str()); ++failures; }
}
const int A = 0, B = 0, C = 0;   // owners
std::string call(Order &o, int device, const void *owner, int st)
{
    done.clear();
    Order::Turn turn(o, device, owner, st);
    return done;
}

void rules()
{
    Order o;
    check(call(o, 0, &A, 10).empty(), "the first call waits for nothing");
    check(call(o, 0, &A, 10).empty() && call(o, 0, &B, 10).empty(), "calls on one stream need no event, whoever makes them");
    check(call(o, 0, &C, 11) == "r10 w11 ", "a call on another stream starts behind the last one");
    check(call(o, 0, &C, 11).empty() && call(o, 0, &A, 10) == "r11 w10 ", "and back");
    check(call(o, 1, &C, 11).empty(), "devices are apart");
    check(call(o, 0, &A, 0) == "r10 w0 " && call(o, 0, &A, 10) == "r0 w10 ", "the default stream is one like the others");
    check(call(o, 0, &C, 2).empty() && call(o, 0, &A, 10).empty(), "a stream per thread is left alone");
    check(call(o, 9, &C, 12).empty() && call(o, -1, &C, 13).empty(), "devices out of range");
}
void captures()
{
    Order o;
    call(o, 0, &A, 10);
    in_capture = {11};
    check(call(o, 0, &C, 11).empty(), "a captured call gets no event");
    check(call(o, 0, &B, 12) == "r10 w12 ", "and is not the one that the next waits for");
    in_capture = {12};
    check(call(o, 0, &A, 10).empty(), "no event on a stream that is being captured");
    in_capture.clear();
    check(call(o, 0, &B, 12) == "r10 w12 ", "the call in between counts");
}
void owners_go()
{
    Order o;
    call(o, 0, &A, 10);
    call(o, 0, &B, 11);
    const int x = 0;
    o.forget(&x);
    check(call(o, 0, &A, 10) == "r11 w10 ", "another owner's end changes nothing");
    o.forget(&A);
    check(events == 0, "its event goes too");
    check(call(o, 0, &B, 11).empty(), "behind the end of the last owner there is nothing to wait for");
    call(o, 0, &A, 66);
    check(call(o, 0, &B, 11) == "r66 ", "a stream that is gone is not waited for");
    o.forget(&B);
    check(events == 0, "no event is left");
}
// one call enqueues at a time
void threads()
{
    Order o;
    std::atomic<int> inside{0};
    std::vector<std::thread> ts;
    std::atomic<bool> ok{true};
    for (int i = 0; i < 8; ++i)
        ts.emplace_back([&, i] {
            static const int owner[8] = {};
            for (int k = 0; k < 2000; ++k) {
                {
                    Order::Turn turn(o, 0, &owner[i], 20 + i % 3);
                    if (inside.fetch_add(1) != 0) ok = false;
                    inside.fetch_sub(1);
                }
                if (k % 100 == 99) o.forget(&owner[i]);
            }
        });
    for (std::thread &t : ts) t.join();
    check(ok, "turns do not overlap");
}
}  // namespace

int main(int argc, char **argv)
{
    if (argc != 2) return 2;
    if (!std::strcmp(argv[1], "rules")) rules();
    else if (!std::strcmp(argv[1], "captures")) captures();
    else if (!std::strcmp(argv[1], "owners_go")) owners_go();
    else if (!std::strcmp(argv[1], "threads")) threads();
    else return 2;
    return failures ? 1 : 0;
}
