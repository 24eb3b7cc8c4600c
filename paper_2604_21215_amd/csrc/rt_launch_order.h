// Order among the calls of a process whose kernels want every compute unit of a device at once because their workgroups wait for one
// another.  On one stream they follow each other; from two streams two such grids could each hold a part of the chip and wait for
// the rest (cooperative launches queue up behind each other, but not behind the ordinary launches of the decoding step and of the
// backward pass's loop).  So a call that comes on another stream than the one before it starts behind what that stream holds.
//
// A program with one stream pays a lock without contention (20 ns); the lock is held while a call enqueues its work, so that an
// event of the next call lies behind all of it.  Left alone are calls on a stream that is being captured, or after one whose stream is
// being captured now (an event would become part of the capture), and hipStreamPerThread, which names a stream per thread.
//
// Api: Stream, Event, per_thread(), capturing(stream), create(), record(event, stream), wait(stream, event), destroy(event): bool where
// they can fail.  Plain host code: the rules are checked without a GPU.
#pragma once
#include <mutex>

namespace rt {

template <class Api, int kDevices = 64> class LaunchOrder {
public:
    using Stream = typename Api::Stream;
    using Event = typename Api::Event;

    // A call of `owner` on `st` enqueues its work while this lives.
    class Turn {
    public:
        Turn(LaunchOrder &order, int device, const void *owner, Stream st) : lock_(order.mu_)
        {
            if (device < 0 || device >= kDevices || st == Api::per_thread()) return;
            Last &l = order.last_[device];
            if (!l.owner || l.stream != st) {
                if (Api::capturing(st)) return;
                if (l.owner && !Api::capturing(l.stream) && (l.has_event || (l.has_event = Api::create(&l.event))) &&
                    Api::record(l.event, l.stream))
                    (void)Api::wait(st, l.event);
            }
            l.owner = owner;
            l.stream = st;
        }

    private:
        std::lock_guard<std::mutex> lock_;
    };

    // `owner` goes, its work is done and its stream may go too
    void forget(const void *owner)
    {
        std::lock_guard<std::mutex> lock(mu_);
        for (Last &l : last_)
            if (l.owner == owner) {
                l.owner = nullptr;
                if (l.has_event) Api::destroy(l.event);
                l.has_event = false;
            }
    }

private:
    struct Last {
        const void *owner = nullptr;   // of the last call, null: none that may still run
        Stream stream{};
        Event event{};
        bool has_event = false;
    };
    std::mutex mu_;
    Last last_[kDevices];
};

}  // namespace rt
