// Waiting on the host for a word that the device writes.
#pragma once

#include <thread>

namespace auxp {

// What to do between two looks at the word: a pause of the core's other
// hardware thread at first, since the next report of a small solve is some
// 30 us away, then the core to whoever else wants it.  (A loop of loads alone
// kept the core for whole time slices: two such threads on one core hand a word
// over in 4 ms instead of 10 us.)
class Polling {
    int turns = 0;

public:
    void pause()
    {
        if (turns < 512) {
            turns++;
            __builtin_ia32_pause();
        } else {
            std::this_thread::yield();
        }
    }
};

}  // namespace auxp
