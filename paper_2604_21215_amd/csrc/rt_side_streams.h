// Side streams of the layer-wavefront engine, lent to a call for the time it enqueues its work and shared by the contexts of a
// process.  A process has four hardware queues and a stream keeps the one it was given: with two side streams per context the
// streams of several contexts share queues with each other and with the caller's stream, and groups of layers that should overlap
// run one after the other (12 layers, B = 4, N = 4096: 285 ms for the only context of a process, 420 - 725 ms for some of several on
// one stream, 284 ms for all of them from here).
//
// A set goes back with work still queued on it, and that work waits for the caller's stream it was lent to.  So it is lent again
// only to a call on the same caller's stream, whose order it shares anyway, or once it has run dry: a call never waits for what another
// stream has queued.  Calls on several threads at once take different sets; there are no more of them than contexts.  hipStreamPerThread names a stream per thread and
// counts as a different one every time.
//
// Api: Stream, per_thread(), idle(stream), destroy(device, stream).  Plain host code: the rules are checked without a GPU.
#pragma once
#include <cstddef>
#include <mutex>
#include <new>

namespace rt {

template <class Api, int kSide> class SidePool {
public:
    using Stream = typename Api::Stream;
    struct Set {
        int device;
        Stream caller;      // of the work that may be queued
        Stream st[kSide];   // created by the call that first needs them
        Set *next;
    };

    // nullptr: out of memory
    Set *take(int device, Stream caller)
    {
        std::lock_guard<std::mutex> lock(mu_);
        Set **found = nullptr;
        for (Set **p = &free_; *p && !found; p = &(*p)->next)
            if ((*p)->device == device && (*p)->caller == caller && caller != Api::per_thread()) found = p;
        for (Set **p = &free_; *p && !found; p = &(*p)->next)
            if ((*p)->device == device && idle(**p)) found = p;
        Set *s = found ? *found : new (std::nothrow) Set{device, caller, {}, nullptr};
        if (found) { *found = s->next; --count_; }
        if (s) s->caller = caller;
        return s;
    }
    void give(Set *s)
    {
        std::lock_guard<std::mutex> lock(mu_);
        s->next = free_;
        free_ = s;
        ++count_;
    }
    // Contexts of the process.  There is never use for more sets than contexts: when one goes, idle sets beyond that number go too
    // (work of other contexts may still be queued on the others), with the last one all of them.
    void count_context(int change)
    {
        Set *gone = nullptr;
        {
            std::lock_guard<std::mutex> lock(mu_);
            contexts_ += change;
            for (Set **p = &free_; change < 0 && *p && count_ > contexts_;) {
                Set *s = *p;
                if (contexts_ > 0 && !idle(*s)) { p = &s->next; continue; }
                *p = s->next;
                --count_;
                s->next = gone;
                gone = s;
            }
        }
        while (gone) {   // outside the lock, and never inside a call that has work queued: giving a stream back may wait for it
            Set *s = gone;
            gone = s->next;
            for (Stream &st : s->st)
                if (st) Api::destroy(s->device, st);
            delete s;
        }
    }

private:
    static bool idle(const Set &s)
    {
        for (const Stream &st : s.st)
            if (st && !Api::idle(st)) return false;
        return true;
    }
    std::mutex mu_;
    Set *free_ = nullptr;
    int count_ = 0, contexts_ = 0;
};

}  // namespace rt
