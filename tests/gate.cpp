// The gate of launches whose workgroups wait for each other (ska_gate.h), on the host.  Prints the first violation and returns 1.
#include "ska_gate.h"

#include <cstdio>

#define MUST(COND)                                          \
    do {                                                    \
        if (!(COND)) {                                      \
            std::printf("line %d: %s\n", __LINE__, #COND);  \
            return 1;                                       \
        }                                                   \
    } while (0)

int main()
{
    int x = 0, y = 0;
    const WaitStream a{&x, {}}, b{&y, {}}, null{};
    unsigned word[2] = {0, 0};
    WaitGate g;
    MUST(!g.may_start(a));   // no memory: nobody could say that it has started
    g.word = word;
    MUST(g.may_start(a) && g.may_start(b) && g.may_start(null));
    // one that has not started yet, of whichever kind: only its own stream goes on
    g.launched(a);
    MUST(g.may_start(a) && !g.may_start(b) && !g.may_start(null));
    g.launched(a);
    word[0] = 1;   // the first has started, the second has not
    MUST(g.may_start(a) && !g.may_start(b));
    word[0] = 2;
    MUST(g.may_start(a) && g.may_start(b) && g.may_start(null));
    g.launched(null);
    MUST(!g.may_start(a) && g.may_start(null));
    word[0] = 3;
    // the per-thread stream: one handle, a stream per thread
    std::thread::id other;
    std::thread t([&] { other = std::this_thread::get_id(); });
    const WaitStream mine{&x, std::this_thread::get_id()}, theirs{&x, t.get_id()};
    t.join();
    MUST(theirs.thread == other);
    g.launched(mine);
    MUST(g.may_start(mine) && !g.may_start(theirs) && !g.may_start(a));
    // a wait that ran out: launches for a while, longer each time that it happens soon again
    word[0] = 4;
    for (unsigned round = 0, length = WaitGate::PAUSE; round < 14; ++round, length = length < WaitGate::LONGEST ? 2 * length : length) {
        MUST(g.may_start(a));
        g.launched(a);
        word[0] = word[1] = g.seq;
        for (unsigned i = 0; i < length; ++i) MUST(!g.may_start(i & 1 ? a : b));
    }
    MUST(g.may_start(a) && g.length == WaitGate::LONGEST);
    // ... and as long as at first after many that went well
    for (unsigned i = 0; i < 64 * WaitGate::LONGEST + 1; ++i) g.launched(a);
    word[0] = word[1] = g.seq;
    MUST(!g.may_start(a) && g.pause == WaitGate::PAUSE - 1);
    g.forget();
    MUST(g.may_start(a));
    // numbers go round
    g.seq = word[0] = ~0u;
    g.launched(b);
    MUST(g.seq == 0 && !g.may_start(a));
    word[0] = 0;
    MUST(g.may_start(a));
    std::printf("ok\n");
    return 0;
}
