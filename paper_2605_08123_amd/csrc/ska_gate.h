// The order of launches whose workgroups wait for each other.  Plain C++.
#pragma once
#include <thread>

namespace {

// A stream as the host tells it from others.  The per-thread stream's handle is the same in every thread.
struct WaitStream {
    const void *handle = nullptr;
    std::thread::id thread;   // of the per-thread stream
    bool operator==(const WaitStream &o) const { return handle == o.handle && thread == o.thread; }
};

// One per device, for both kinds of such launches: chains of whole steps (vstep_kernel) and of half-steps (vchain_kernel).  Two that
// are placed in part hold each other's workgroups out.  So one starts only behind the latest on the same stream, or
// after all workgroups of the latest have started, which then need nothing more (and so did those of all before it).  Otherwise the
// caller launches steps or half-steps one by one, with the same results.  (g_mutex held)
struct WaitGate {
    unsigned *word = nullptr, *word_dev = nullptr;   // host memory that the device writes: numbers of the latest launch that has started
                                                     // as a whole, of the latest in which a wait has run out
    unsigned seq = 0;                                // number of the latest launch
    unsigned goal = 0;                               // workgroups of all chains of half-steps so far (they are counted by one word)
    WaitStream last;
    unsigned started() const { return word ? __atomic_load_n(word, __ATOMIC_RELAXED) : 0u; }
    unsigned given_up() const { return word ? __atomic_load_n(word + 1, __ATOMIC_RELAXED) : 0u; }
    bool may_start(const WaitStream &s) const { return word && (started() == seq || (seq && s == last)); }
    void launched(const WaitStream &s) { ++seq; last = s; }
};

}  // namespace
