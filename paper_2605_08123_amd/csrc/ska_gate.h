// The order of launches whose workgroups wait for each other.  Plain C++.
#pragma once
#include <thread>

namespace {

// A stream as the host tells it from others.  The per-thread stream's handle is the same in every thread.  (A new stream that gets a
// destroyed one's handle passes for it; if the latest launch still waits for room then, the two may run out of their waits.)
struct WaitStream {
    const void *handle = nullptr;
    std::thread::id thread;   // of the per-thread stream
    bool operator==(const WaitStream &o) const { return handle == o.handle && thread == o.thread; }
};

// One per device, for both kinds of such launches: chains of whole steps (vstep_kernel) and of half-steps (vchain_kernel).  Two that
// are placed in part hold each other's workgroups out.  So one starts only behind the latest on the same stream, or
// after all workgroups of the latest have started, which then need nothing more (and so did those of all before it).  Otherwise the
// caller launches steps or half-steps one by one, with the same results.
//   (A stream whose kernels do not run on all CUs has no such launches: what fits the device may not fit those.)
//   A wait that runs out means that something this process does not know of keeps workgroups out (another program, a kernel that stays),
// and costs a call a tenth of a second and the solve anew.  So the calls after it are launched: PAUSE of them, twice as many each
// time that it happens soon again.  (g_mutex held)
struct WaitGate {
    unsigned *word = nullptr, *word_dev = nullptr;   // host memory that the device writes: numbers of the latest launch that has started
                                                     // as a whole, of the latest in which a wait has run out
    unsigned seq = 0;                                // number of the latest launch
    unsigned goal = 0;                               // workgroups of all chains of half-steps so far (they are counted by one word)
    unsigned seen = 0, length = 0, pause = 0;        // given_up() as last looked at; calls to be launched after it, and of those still
    WaitStream last;
    static constexpr unsigned PAUSE = 256, LONGEST = 1u << 20;
    unsigned started() const { return word ? __atomic_load_n(word, __ATOMIC_RELAXED) : 0u; }
    unsigned given_up() const { return word ? __atomic_load_n(word + 1, __ATOMIC_RELAXED) : 0u; }
    bool may_start(const WaitStream &s)
    {
        const unsigned gave = given_up();
        if (gave != seen) {
            const bool soon = length && gave - seen <= 64 * length;
            length = !soon ? PAUSE : length < LONGEST ? 2 * length : length;
            pause = length;
            seen = gave;
        }
        if (pause) {
            --pause;
            return false;
        }
        return word && (started() == seq || (seq && s == last));
    }
    void forget() { seen = given_up(); length = pause = 0; }
    void launched(const WaitStream &s) { ++seq; last = s; }
};

}  // namespace
