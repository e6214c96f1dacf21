// Phase timings of a solve: stamps of the device's clock in pinned host memory,
// written by the stream at the phases' ends and read when the host has waited
// for the stream anyway.  Host code only.
#pragma once

#include <vector>

namespace dd {

enum { CLOCK_SLOTS = 64 };

// Device: stamp(p) enqueues the writing of the device's clock to *p, wait()
// waits for everything enqueued, ms_per_tick() is the clock's tick.
//
// Stamps are numbered in the order they are taken; stamp i lies in slot i mod
// CLOCK_SLOTS until it is read, and no slot is used again before that.  What
// has been read is kept for 2 CLOCK_SLOTS stamps more, so the start of a span
// still open when the slots are read is not lost.
template <typename Device> struct Clock {
    struct Span {
        long a, b;
        double *acc;
    };
    Device dev;
    unsigned long long *const t;                 // [CLOCK_SLOTS]
    unsigned long long tick[2 * CLOCK_SLOTS];    // stamps read
    std::vector<Span> spans;                     // closed and not yet added up
    long n = 0, read = 0, last_end = -1;
    Clock(const Device &d, unsigned long long *slots) : dev(d), t(slots) {}
    unsigned long long *at(long i) const { return t + i % CLOCK_SLOTS; }
    // A stamp that a kernel writes to *at(i), enqueued before the next stamp.
    long slot()
    {
        if (n - read == CLOCK_SLOTS) finish();
        return n++;
    }
    long mark()
    {
        const long i = slot();
        dev.stamp(at(i));
        return i;
    }
    void add(long a, long b, double *acc)
    {
        spans.push_back({a, b, acc});
        last_end = b;
    }
    // The stream has been waited for since the last stamp.
    void collect()
    {
        for (; read < n; read++) tick[read % (2 * CLOCK_SLOTS)] = *at(read);
        for (const Span &p : spans)
            *p.acc += (double)(long long)(tick[p.b % (2 * CLOCK_SLOTS)] - tick[p.a % (2 * CLOCK_SLOTS)]) * dev.ms_per_tick();
        spans.clear();
    }
    void finish()
    {
        dev.wait();
        collect();
    }
};

// A span from construction to destruction; follows: it starts where the span
// added last ended (nothing was launched since).
template <typename Device> struct Timer {
    Clock<Device> &clk;
    double *acc;
    long a;
    Timer(Clock<Device> &c, double *acc_, bool follows = false)
        : clk(c), acc(acc_), a(follows && c.last_end >= 0 ? c.last_end : c.mark())
    {
    }
    ~Timer() { clk.add(a, clk.mark(), acc); }
};

}  // namespace dd
